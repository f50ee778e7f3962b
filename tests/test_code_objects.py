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
def objects(tmp_path_factory):
    """the library's gfx950 code objects, as files"""
    blob, magic, files = build.LIB.read_bytes(), b"__CLANG_OFFLOAD_BUNDLE__", []
    at, tmp = blob.find(magic), tmp_path_factory.mktemp("code")
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        entry = at + len(magic) + 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, entry)
            name = blob[entry + 24:entry + 24 + name_len].decode()
            entry += 24 + name_len
            if "gfx950" not in name or not size:
                continue
            files.append(tmp / f"object{len(files)}.elf")
            files[-1].write_bytes(blob[at + offset:at + offset + size])
        at = blob.find(magic, at + 1)
    return files


@pytest.fixture(scope="module")
def kernels(objects):
    """{mangled name: {"vgprs", "spilled", "scratch"}} of every kernel of the library"""
    found = {}
    for path in objects:
        notes = subprocess.run([str(READELF), "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for part in notes.split("  - .agpr_count:")[1:]:
            def number(key):
                return int(re.search(rf"\.{key}:\s+(\d+)", part)[1])
            found[re.search(r"\.name:\s+(\S+)", part)[1]] = {
                "vgprs": number("vgpr_count"), "spilled": number("vgpr_spill_count"), "scratch": number("private_segment_fixed_size")}
    assert len(found) > 50
    return found


@pytest.fixture(scope="module")
def code(objects):
    """{mangled name: its instructions, one a line}"""
    found = {}
    for path in objects:
        text = subprocess.run([str(READELF.with_name("llvm-objdump")), "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            name, _, body = part.partition(">:")
            found[name] = body
    return found


def pick(kernels, pattern, count):
    got = {name: k for name, k in kernels.items() if re.search(pattern, name)}
    assert len(got) == count, (pattern, list(got))
    return got


def test_staged_generic_gemms_keep_their_workgroups_a_cu(kernels):
    # four epilogues each; registers of a wave, accumulators among them: 512 / 3 with three workgroups of four waves to a CU, 512 / 2 else
    for pattern, vgprs in ((r"12k_plain_gemmItLi\dELi4ELi4ELi2ELi2ELi1ELi1ELi3E", 168), (r"12k_plain_gemmItLi\dELi2ELi4ELi4ELi2ELi1ELi1ELi4E", 256),
                           (r"12k_plain_gemmIfLi\dELi2ELi4ELi4ELi2ELi1ELi2ELi2E", 256), (r"12k_plain_gemmI[ft]Li\dELi2ELi2ELi2ELi2ELi2ELi1ELi4E", 256)):
        for name, k in pick(kernels, pattern, 8 if "[ft]" in pattern else 4).items():
            assert k["vgprs"] <= vgprs and k["spilled"] == 0 and k["scratch"] == 0, (name, k)


def test_decode_attention_keeps_two_waves_a_simd(kernels):
    # chunked: called directly and recorded; short: one block ahead (four waves a SIMD) and two, with and without reading ahead
    for pattern, count, vgprs in ((r"13k_attn_decodeILb", 2, 256), (r"19k_attn_decode_shortILi1E", 2, 128), (r"19k_attn_decode_shortILi2E", 2, 256)):
        for name, k in pick(kernels, pattern, count).items():
            assert k["vgprs"] <= vgprs and k["spilled"] == 0 and k["scratch"] == 0, (name, k)


def test_prefill_gemms_do_not_spill(kernels):
    # five pairs of epilogue and class in three forms; the wide one (waves 4 x 2, four token blocks each) keeps 8 waves a CU
    for name, k in pick(kernels, r"6k_gemmILi\dELi\dENS0_8GemmForm", 15).items():
        assert k["vgprs"] <= 256 and k["spilled"] == 0 and k["scratch"] == 0, (name, k)


def test_generic_decode_contractions_do_not_spill(kernels):
    # float and bf16; up to 4, 8, 16, 32 tokens in 8 and 16 waves; four epilogues, and the opening form of QKV up to 8 tokens
    for name, k in pick(kernels, r"12k_plain_gemvI[ft]L", 2 * 2 * (4 * 4 + 2)).items():
        assert k["spilled"] == 0 and k["scratch"] == 0, (name, k)


def test_generic_decode_attention_does_not_spill(kernels):
    for name, k in (pick(kernels, r"16k_plain_dec_attnI[ft]L", 10) | pick(kernels, r"22k_plain_dec_attn_partsI[ft]L", 4)).items():
        assert k["spilled"] == 0 and k["scratch"] == 0, (name, k)


def test_decode_gemvs_do_not_spill_and_one_window_is_built_where_a_plan_has_one(kernels):
    # (epilogue, row blocks, waves, class): QKV and the opening one in three forms, gate/up in one, O, down and the last down in two
    in_several, in_one = (pick(kernels, rf"10k_dec_gemvILi\dELi\dELi\dELi\d+ELb{short}EE", count) for short, count in ((0, 13), (1, 8)))
    for name, k in (in_several | in_one).items():
        assert k["spilled"] == 0 and k["scratch"] == 0, (name, k)
        assert k["vgprs"] <= (256 if name in in_one or "k_dec_gemvILi4E" in name else 128), (name, k)  # waves a SIMD: two, four


# The last workgroup of a split row group or tile to arrive reads what the others have stored in the same launch: at device scope (sc1), as
# they stored it, or a line that its L2 has kept from an earlier launch could answer.
@pytest.mark.parametrize("pattern,count", [
    (r"10k_dec_gemvILi1ELi2ELi8ELi10ELb0EE", 1), (r"10k_dec_gemvILi[23]ELi2ELi8ELi(9|12)ELb0EE", 3),  # gate/up; O, down and the last down
    (r"6k_gemmILi\dELi\dENS0_8GemmFormILi\dELi\dELi[12]E", 10)])                                             # the prefill forms of up to 128 tokens
def test_partial_sums_of_other_workgroups_are_read_at_device_scope(code, pattern, count):
    for name, text in pick(code, pattern, count).items():
        lines = [line for line in text.splitlines() if " sc1" in line.split("//")[0]]
        stores, loads = ([line for line in lines if f"global_{what}_dword" in line] for what in ("store", "load"))
        assert stores and len(loads) >= 16, (name, len(stores), len(loads))
