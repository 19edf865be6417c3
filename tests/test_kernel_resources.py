"""What the launchers take for granted about the compiled kernels, read from the metadata of the code objects in
libfbq.so (built here from csrc/): registers, spills and LDS of every instance."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

import paper_2501_16385_amd as fbq


def code_objects():
    """The metadata of every kernel: the AMDGPU notes of the ELF images inside the library."""
    data, found, pos = open(fbq.lib_path(), "rb").read(), [], 0
    while (i := data.find(b"\x7fELF", pos)) >= 0:
        pos = i + 4
        if struct.unpack_from("<H", data, i + 18)[0] != 224:        # EM_AMDGPU
            continue
        table, = struct.unpack_from("<Q", data, i + 40)
        entry, count = struct.unpack_from("<HH", data, i + 58)
        for s in range(count):
            kind, = struct.unpack_from("<I", data, i + table + s * entry + 4)
            offset, size = struct.unpack_from("<QQ", data, i + table + s * entry + 24)
            p, end = i + offset, i + offset + size
            while kind == 7 and p < end:                            # SHT_NOTE
                name, desc, _ = struct.unpack_from("<III", data, p)
                d = p + 12 + (name + 3 & ~3)
                if data[p + 12:p + 12 + name] == b"AMDGPU\0":
                    found += msgpack.unpackb(data[d:d + desc])["amdhsa.kernels"]
                p = d + (desc + 3 & ~3)
    return found


@pytest.fixture(scope="module")
def kernels():
    found = code_objects()
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), text=True, capture_output=True, check=True).stdout.split("\n")
    return {re.sub(r"^void |\(.*", "", n): k for n, k in zip(names, found)}


def test_two_blocks_of_the_gemv_fit_a_compute_unit(kernels):
    """launch_gemv_decode hands out two blocks of four waves per CU with fixed tile lists and counts on all of them being
    resident: two waves per SIMD, i.e. at most 256 of its 512 registers each, and half of the 160 KiB of LDS."""
    gemv = {n: k for n, k in kernels.items() if "fbq_gemv_kernel<" in n}
    assert len(gemv) >= 54                                          # 2 bit widths x 9 shapes x 3 rank classes
    for n, k in gemv.items():
        assert k[".vgpr_count"] <= 256 and k[".vgpr_spill_count"] == 0, n
        assert k[".group_segment_fixed_size"] <= 80 * 1024, n


def test_streaming_instances_have_their_registers_and_a_cu_each(kernels):
    """One block of eight waves per CU: two waves per SIMD, 256 registers each, no scratch memory (that alone costs a launch 2 us; scalar registers do spill
    into vector ones), and more than half of the LDS, so that no second block starts beside it on rows that were meant for another CU."""
    stream = {n: k for n, k in kernels.items() if "fbq_few_stream_kernel<" in n}
    assert len(stream) == 24                                        # 2 bit widths x 3 shapes of K x 2 token classes x (in a grid, in line)
    for n, k in stream.items():
        assert k[".vgpr_count"] <= 256 and k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, n
        assert 80 * 1024 < k[".group_segment_fixed_size"] <= 160 * 1024, n


def test_split_instances_have_their_registers_and_a_cu_each(kernels):
    """As the streaming kernel's: two waves per SIMD without scratch memory, and more than half of the LDS, since the plan counts one block per CU."""
    split = {n: k for n, k in kernels.items() if "fbq_few_split_kernel<" in n}
    assert len(split) == 10                                         # 2 bit widths x (1 set of up to 8 and up to 16 tokens, 2, 3, 4 sets)
    for n, k in split.items():
        assert k[".vgpr_count"] <= 256 and k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, n
        assert 80 * 1024 < k[".group_segment_fixed_size"] <= 160 * 1024, n


def test_quantizer_instances_have_their_registers(kernels):
    """No scratch memory, and the waves a SIMD that the launch bounds ask for wherever the LDS allows them: four without Delta_F, three with (two above rank 128)."""
    quant = {n: k for n, k in kernels.items() if "fbq_quantize_kernel<" in n}
    assert len(quant) == 22                                         # 2 bit widths x (4 shapes with and without Delta_F, 3 in fp64 with it)
    for n, k in quant.items():
        delta, steps, waves = re.search(r"<\d, (\w+), (\d), (\d)", n).groups()
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, n
        blocks = 160 * 1024 // k[".group_segment_fixed_size"]       # of `waves` waves on four SIMDs
        wanted = min(blocks * int(waves) // 4, 4 if delta == "false" else 2 if steps == "8" else 3)
        assert k[".vgpr_count"] <= 512 // wanted // 8 * 8, (n, k[".vgpr_count"], wanted)


def test_inline_assembly_declares_the_scalar_register_it_overwrites():
    """M0 belongs to the compiler: a statement that moves an LDS address into it without saying so would silently change
    whatever value the compiler keeps there."""
    csrc = os.path.join(os.path.dirname(fbq.lib_path()), "csrc")
    found = 0
    for name in sorted(os.listdir(csrc)):
        for statement in re.findall(r"\basm\b[^;]*;", open(os.path.join(csrc, name)).read()):
            if re.search(r"\bs_mov_b32 m0\b", statement):
                found += 1
                assert statement.rstrip(");").endswith('"m0"'), (name, statement)
    assert found == 3
