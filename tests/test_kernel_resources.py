"""CPU-only checks of the kernels' registers: none spilled to scratch, and no more than leave the wavefronts room that a
launch needs to hide its loads."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2207_02849_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_vector_kernels_do_not_spill(tmp_path):
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(build.CSRC, "kernels.hip"), "-o", str(tmp_path / "kernels.o")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+).*?VGPRs Spill: (\d+)", r.stderr, flags=re.S)
    assert any("last_layer_rop" in k for k, _, _ in kernels)
    spilled = [k for k in kernels if k[1] != "0" or k[2] != "0"]
    assert not spilled, spilled


def built_kernels():
    """{name: metadata} of the kernels in the built library: the notes of its code objects (one bundle a source)."""
    data, found = open(build.LIB, "rb").read(), {}
    for bundle in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        count, at = struct.unpack_from("<Q", data, bundle.start() + 24)[0], bundle.start() + 32
        for _ in range(count if count < 16 else 0):
            offset, size, n = struct.unpack_from("<QQQ", data, at)
            target, at = data[at + 24:at + 24 + n], at + 24 + n
            if b"amdgcn" not in target or not size:
                continue
            elf = data[bundle.start() + offset:bundle.start() + offset + size]
            sections, (entry, number) = struct.unpack_from("<Q", elf, 0x28)[0], struct.unpack_from("<HH", elf, 0x3A)
            for header in range(sections, sections + number * entry, entry):
                start, length = struct.unpack_from("<QQ", elf, header + 24)
                while struct.unpack_from("<I", elf, header + 4)[0] == 7 and length > 0:       # SHT_NOTE
                    name, desc, kind = struct.unpack_from("<III", elf, start)
                    body, step = start + 12 + (name + 3) // 4 * 4, 12 + (name + 3) // 4 * 4 + (desc + 3) // 4 * 4
                    if kind == 32:                                                            # NT_AMDGPU_METADATA
                        found.update((k[".name"], k) for k in msgpack.unpackb(elf[body:body + desc], strict_map_key=False)["amdhsa.kernels"])
                    start, length = start + step, length - step
    return found


@pytest.mark.skipif(not os.path.exists(build.LIB), reason="not built")
def test_forward_kernels_leave_four_wavefronts_a_simd():
    """512 registers a SIMD lane: forward products on 64-tiles and 128 x 64 tiles (epilogue modes 1 and 2) within 128.  With 140 a
    forward product of 27068 samples between 97-wide layers took 19.1 us, with 124 14.7."""
    forward = {k: m for k, m in built_kernels().items()
               if re.search(r"gemm_fused_kernelI(DF16b|f)Li(64ELi64ELi8ELi4|128ELi64ELi8ELi8)ELi1ELi[12]E", k)}
    assert len(forward) == 8
    crowded = {k: m[".vgpr_count"] for k, m in forward.items() if m[".vgpr_count"] > 128 or m[".vgpr_spill_count"]}
    assert not crowded, crowded


@pytest.mark.skipif(not os.path.exists(build.LIB), reason="not built")
def test_no_kernel_keeps_arrays_in_scratch():
    """(An epilogue too large for its tile's registers had 1344 bytes a lane there: up to 1.25 times the time of a call.)"""
    kernels = built_kernels()
    assert len(kernels) > 300
    scratch = {k: m[".private_segment_fixed_size"] for k, m in kernels.items() if m[".private_segment_fixed_size"] or m[".vgpr_spill_count"]}
    assert not scratch, scratch
