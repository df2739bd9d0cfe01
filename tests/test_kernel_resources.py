"""What the built kernels take of a CU, from the metadata of the library's own gfx950 code objects (no GPU needed)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name: (VGPRs, bytes of scratch per lane)} of every kernel in libvcas.so."""
    from paper_2402_17227_amd import binding, build
    if not os.path.exists(os.path.join(LLVM, "llvm-readelf")) or not shutil.which("c++filt"):
        pytest.skip("needs the LLVM tools the library is built with")
    if not os.path.exists(binding.LIB_PATH):
        build.build(force=True)
    tmp = tmp_path_factory.mktemp("code")
    fat = tmp / "fat.bin"
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", binding.LIB_PATH, str(tmp / "copy.so")],
                   check=True)
    data, found, at = fat.read_bytes(), {}, 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entries, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" not in target or not size:
                continue
            obj = tmp / "one.co"
            obj.write_bytes(data[at + offset:at + offset + size])
            notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
            for block in notes.split("  - .agpr_count:")[1:]:
                field = lambda key: re.search(rf"\.{key}:\s+(\S+)", block).group(1)
                name = subprocess.run(["c++filt", field("name")], check=True, capture_output=True, text=True).stdout.strip()
                found[name] = (int(field("vgpr_count")), int(field("private_segment_fixed_size")))
        at += 24
    assert found
    return found


def test_256x256_dgrad_leaves_registers_for_side_streams(kernels):
    """Eight wavefronts of it are two to a SIMD of 512 VGPRs: at 224 each there is room for the wavefronts of the norm
    passes (at most 64 VGPRs) that a stack's other streams run beside it, above that (allocation is by 8) for fewer and
    at 248 for none."""
    big = {n: r for n, r in kernels.items() if re.search(r"dgrad_bf16(_group)?_kernel<256, 256", n)}
    assert len(big) == 2
    for name, (vgprs, scratch) in big.items():
        assert vgprs <= 224 and scratch == 0, (name, vgprs, scratch)
