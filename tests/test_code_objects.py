"""What the compiler made of the kernels, read from the metadata of the code objects in the built library: registers (which
decide how many waves share a SIMD of 512) and scratch memory of the kernels whose speed rests on them."""
import pathlib
import re
import struct
import subprocess

import pytest

from paper_2511_14450_amd import build

READELF = pathlib.Path(build.HIPCC).resolve().parents[1] / "llvm" / "bin" / "llvm-readelf"
if not READELF.exists():
    READELF = pathlib.Path("/opt/rocm/llvm/bin/llvm-readelf")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: {"vgprs", "spilled", "scratch"}} of every kernel of the library"""
    blob, magic, found = build.LIB.read_bytes(), b"__CLANG_OFFLOAD_BUNDLE__", {}
    at, tmp = blob.find(magic), tmp_path_factory.mktemp("code") / "object.elf"
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        entry = at + len(magic) + 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, entry)
            name = blob[entry + 24:entry + 24 + name_len].decode()
            entry += 24 + name_len
            if "gfx950" not in name or not size:
                continue
            tmp.write_bytes(blob[at + offset:at + offset + size])
            notes = subprocess.run([str(READELF), "--notes", str(tmp)], capture_output=True, text=True, check=True).stdout
            for part in notes.split("  - .agpr_count:")[1:]:
                def number(key):
                    return int(re.search(rf"\.{key}:\s+(\d+)", part)[1])
                found[re.search(r"\.name:\s+(\S+)", part)[1]] = {
                    "vgprs": number("vgpr_count"), "spilled": number("vgpr_spill_count"), "scratch": number("private_segment_fixed_size")}
        at = blob.find(magic, at + 1)
    assert len(found) > 50
    return found


def pick(kernels, pattern, count):
    got = {name: k for name, k in kernels.items() if re.search(pattern, name)}
    assert len(got) == count, (pattern, list(got))
    return got


def test_wide_bf16_generic_gemms_keep_two_waves_a_simd(kernels):
    # four epilogues; registers of a wave, accumulators among them: 512 / 2
    for name, k in pick(kernels, r"12k_plain_gemmItLi\dELi4ELi4ELi2ELi2ELi1E", 4).items():
        assert k["vgprs"] <= 256 and k["scratch"] == 0, (name, k)


def test_prefill_gemms_do_not_spill(kernels):
    # five pairs of epilogue and class in three forms; the wide one (waves 4 x 2, four token blocks each) keeps 8 waves a CU
    for name, k in pick(kernels, r"6k_gemmILi\dELi\dENS0_8GemmForm", 15).items():
        assert k["vgprs"] <= 256 and k["spilled"] == 0 and k["scratch"] == 0, (name, k)


def test_generic_decode_contractions_do_not_spill(kernels):
    # float and bf16; up to 4, 8, 16, 32 tokens in 8 and 16 waves; four epilogues, and the opening form of QKV up to 8 tokens
    for name, k in pick(kernels, r"12k_plain_gemvI[ft]L", 2 * 2 * (4 * 4 + 2)).items():
        assert k["spilled"] == 0 and k["scratch"] == 0, (name, k)


def test_generic_decode_attention_does_not_spill(kernels):
    for name, k in pick(kernels, r"16k_plain_dec_attnI[ft]L", 10).items():
        assert k["spilled"] == 0 and k["scratch"] == 0, (name, k)
