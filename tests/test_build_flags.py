"""What the build flags promise, checked on the generated gfx950 assembly of this library's own kernels (CPU only:
hipcc cross-compiles): no packed-fp32 arithmetic instruction in any kernel, and no fused multiply-add beyond the
ones the sources write out (-ffp-contract=off)."""
import os
import re
import subprocess

import pytest

from paper_2506_17615_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def device_asm(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc is not installed here")
    out = tmp_path_factory.mktemp("asm")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    text = {}
    for src in build.SOURCES:
        dst = out / (os.path.basename(src) + ".s")
        subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", src, "-o", str(dst)], check=True, capture_output=True)
        text[os.path.basename(src)] = dst.read_text()
    return text


def test_no_packed_fp32_arithmetic(device_asm):
    for name, asm in device_asm.items():
        assert ".amdgcn_target" in asm and "gfx950" in asm, name
        packed = re.findall(r"^\s*(v_pk_(?:add|mul|fma)_f32)\b", asm, flags=re.M)
        assert not packed, f"{name}: {len(packed)} packed fp32 instructions"


def test_kernels_are_there_and_use_what_the_sources_say(device_asm):
    asm = device_asm["equarx_api.hip"]
    # the hop kernel of the benchmark's block size exists, widens int8 with byte-select converts, exchanges lanes
    # with DPP and the row swaps, and converts to bf16 in hardware where it writes bf16
    assert re.search(r"^_ZN6equarx10hop_kernelILi256ELi\d+ELb[01]EEEv", asm, flags=re.M)
    assert "v_permlane32_swap" in asm and "v_permlane16_swap" in asm and "row_mirror" in asm
    assert "v_cvt_pk_bf16_f32" in asm
    assert "v_perm_b32" in asm


def test_leading_kernel_arguments_are_preloaded(device_asm):
    asm = device_asm["equarx_api.hip"]
    for kernel, dwords in (("hop_kernelILi256E", 14), ("quantize_kernelILi256E", 10), ("dequantize_kernelILi256E", 10),
                           ("chain_kernelILi256E", 14), ("flat_kernelILi256E", 14)):
        found = re.findall(r"^\s*\.amdhsa_kernel _ZN6equarx\d+" + kernel + r".*?preload_length (\d+)", asm, flags=re.M | re.S)
        assert found and all(int(f) == dwords for f in found), (kernel, found)


def test_the_tiles_of_a_thread_at_the_end_are_requested_together(device_asm):
    """A thread with several tiles waits for none of them before it has asked for all: in the workgroup that holds the
    end of a tensor (the buffer loads) no wait stands between two requests of one straight run of instructions."""
    bodies = re.findall(r"^(_ZN6equarx\d+(?:(?:quantize|hop|dequantize|head|tail)_kernelILi\d+ELi2E|"
                        r"(?:chain|semi)_kernelILi\d+ELi\d+ELi[24]E)\S*):(.*?)^\.Lfunc_end",
                        device_asm["equarx_api.hip"], flags=re.M | re.S)
    assert len({name.split("ILi")[0] for name, _ in bodies}) == 7
    for name, body in bodies:
        requested = waited = False
        for line in body.splitlines():
            if re.match(r"\.L|\s+s_c?branch", line):
                requested = waited = False
            elif "buffer_load" in line:
                assert not waited, name
                requested = True
            elif "vmcnt" in line:
                waited = requested


def test_the_small_kernel_takes_its_partials_without_a_loop(device_asm):
    """All partials of a call are one request unless there are more than 16: no loop, whose every step would ask whether it
    is the first; or unless 9 to 16 keep their wire, which is faster in one."""
    bodies = re.findall(r"^(_ZN6equarx\d+small_kernelILi\d+ELi[48]ELi(8|16)ELb([01])E(?:Lb[01]E){3}Lb([01])E\S*):(.*?)^\.Lfunc_end",
                        device_asm["equarx_api.hip"], flags=re.M | re.S)
    assert {many for _, _, many, _, _ in bodies} == {"0", "1"}
    for name, count, many, wire, body in bodies:
        assert ("Loop Header" in body) == (many == "1" or (count, wire) == ("16", "1")), name


def test_the_loop_of_the_128_chunk_chain_keeps_its_alignment(device_asm):
    for ag in "01":
        body = re.search(r"^_ZN6equarx\d+chain_strided_kernelILi8ELi2ELi8ELb0ELb1ELb" + ag + r"E\S*:(.*?)^\.Lfunc_end",
                         device_asm["equarx_api.hip"], flags=re.M | re.S).group(1)
        assert len(re.findall(r"\.p2align\s+3\n", body)) == 1


def test_a_wire_that_leaves_is_stored_with_its_hint(device_asm):
    """The per-step kernels' code stores, of whole tiles and of the end of a message, are non-temporal at every shape."""
    bodies = re.findall(r"^(_ZN6equarx\d+(?:(?:quantize|hop|quantize_batch)_kernelILi\d+ELi[12]ELb1E|"
                        r"flat_kernelILi\d+ELi[12]ELi\dELb[01]ELb1ELb1ELb1E)\S*):(.*?)^\.Lfunc_end",
                        device_asm["equarx_api.hip"], flags=re.M | re.S)
    assert len(bodies) == 5 * (3 * 2 + 2 * 4)
    for name, body in bodies:
        stores = [line for line in body.splitlines() if re.search(r"(global|buffer)_store_dwordx2", line)]
        assert len(stores) >= 2 and all(line.split(";")[0].rstrip().endswith(" nt") for line in stores), name


def test_no_store_of_16_bytes_takes_an_offset_from_a_scalar_register(device_asm):
    """The next instructions may overwrite what such a store is still reading: its row belongs in the descriptor."""
    for name, asm in device_asm.items():
        stores = re.findall(r"buffer_store_dwordx[34] [^;\n]*", asm)
        assert name != "equarx_api.hip" or stores
        assert not [line for line in stores if re.search(r"\], s\d+ ", line)], name


def _row_is_a_constant(store):
    """Whether the operand behind the descriptor of a buffer store is a constant; anything else is a scalar register."""
    return re.search(r"\bs\[\d+:\d+\],\s*(?:-?\d+|0x[0-9a-f]+)(?=\s|$)", store) is not None


def test_every_wide_store_has_a_constant_behind_its_descriptor(device_asm):
    """As above, with every form that the operand can take: without modifiers behind it, and in m0, vcc or a trap register."""
    for good in ("v[0:3], v4, s[8:11], 0 offen nt", "v[0:3], off, s[8:11], 0", "v[0:3], v4, s[8:11], -1 offen", "v[0:2], off, s[0:3], 64 offset:16"):
        assert _row_is_a_constant("buffer_store_dwordx4 " + good), good
    for bad in ("s20", "m0", "vcc_lo", "ttmp4"):
        for form in ("v[0:3], off, s[8:11], %s", "v[0:3], v4, s[8:11], %s offen nt", "v[0:3], off, s[8:11], %s offset:16"):
            assert not _row_is_a_constant("buffer_store_dwordx4 " + form % bad), (form, bad)
    for name, asm in device_asm.items():
        stores = re.findall(r"buffer_store_(?:dwordx[34]|format_xyzw?|b96|b128)\s[^;\n]*", asm)
        assert name != "equarx_api.hip" or len(stores) > 100
        assert not [line for line in stores if not _row_is_a_constant(line)], name
