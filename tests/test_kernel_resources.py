"""What the built kernels take of a CU and where they wait, from the metadata and the assembly of the library's own gfx950
code objects (no GPU needed)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """The gfx950 code objects of libvcas.so, as files."""
    from paper_2402_17227_amd import binding, build
    if not os.path.exists(os.path.join(LLVM, "llvm-readelf")) or not shutil.which("c++filt"):
        pytest.skip("needs the LLVM tools the library is built with")
    if not os.path.exists(binding.LIB_PATH):
        build.build(force=True)
    tmp = tmp_path_factory.mktemp("code")
    fat = tmp / "fat.bin"
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", binding.LIB_PATH, str(tmp / "copy.so")],
                   check=True)
    data, found, at = fat.read_bytes(), [], 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entries, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" not in target or not size:
                continue
            found.append(tmp / f"{len(found)}.co")
            found[-1].write_bytes(data[at + offset:at + offset + size])
        at += 24
    assert found
    return found


def _demangled(name):
    return subprocess.run(["c++filt", name], check=True, capture_output=True, text=True).stdout.strip()


@pytest.fixture(scope="module")
def kernels(objects):
    """{demangled name: (VGPRs, bytes of scratch per lane)} of every kernel."""
    found = {}
    for obj in objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
        for block in notes.split("  - .agpr_count:")[1:]:
            field = lambda key: re.search(rf"\.{key}:\s+(\S+)", block).group(1)
            found[_demangled(field("name"))] = (int(field("vgpr_count")), int(field("private_segment_fixed_size")))
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


def test_gemms_that_share_a_cu_do_not_spill(objects, kernels):
    """The staged and split weight gradients, the fp32 dgrads and the kernels of both halves: registers for as many wavefronts as their
    tiles want to a SIMD (of 512 VGPRs), none in scratch.  64x128 tiles of dgrad, two workgroups of eight wavefronts to a CU, keep
    two registers there, which no loop with matrix instructions touches."""
    wanted = {"wgrad_staged_kernel<": 128, "wgrad_split_kernel<": 256, "layer_bf16_kernel<": 256, "layer_f32_kernel<": 256,
              "dgrad_f32_kernel<": 256, "dgrad_f32_wide_kernel<128, 128": 256, "dgrad_f32_wide_kernel<64, 128": 128}
    for part, most in wanted.items():
        some = {n: r for n, r in kernels.items() if part in n}
        assert some, part
        for name, (vgprs, scratch) in some.items():
            assert vgprs <= most and scratch <= (16 if "wide_kernel<64, 128" in part else 0), (name, vgprs, scratch)
    seen = 0
    for obj in objects:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True,
                              text=True).stdout
        for body in re.split(r"\n(?=[0-9a-f]+ <)", text):
            if "dgrad_f32_wide_kernelILi64ELi128" not in body.split("\n", 1)[0]:
                continue
            code = [(int(m.group(3), 16), m.group(1), m.group(2))
                    for m in re.finditer(r"^\s+(\S+)(.*?)//\s*([0-9A-F]+):", body, re.M)]
            for at, op, args in code:
                if not op.startswith(("s_cbranch", "s_branch")):
                    continue
                words = int(args.split()[0])
                to = at + 4 + 4 * (words - 65536 if words > 32767 else words)
                loop = [o for a, o, _ in code if to <= a <= at]
                if to <= at and any("mfma" in o for o in loop):
                    assert not any(o.startswith("scratch_") for o in loop), hex(to)
                    seen += 1
    assert seen >= 2      # the loop of whole steps and that of the last ones


def test_fp32_dgrad_gives_a_stage_back_when_it_has_been_read(objects):
    """Behind a barrier of the main loop the next loads go into the stage of the step before: at every barrier of the
    LDS-direct fp32 dgrad kernels the wavefront's own LDS reads have been waited for in so many words, not only because the
    matrix instructions that use them happen to come first."""
    seen = 0
    for obj in objects:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True,
                              text=True).stdout
        for body in re.split(r"\n(?=[0-9a-f]+ <)", text):
            if "dgrad_f32_kernel" not in body.split("\n", 1)[0]:
                continue
            code = [line.split("//")[0].strip() for line in body.split("\n")[1:]]
            code = [c for c in code if c]
            barriers = [i for i, c in enumerate(code) if c.startswith("s_barrier")]
            assert barriers
            for i in barriers:
                j = i - 1
                while code[j].startswith("s_waitcnt") and "lgkmcnt(0)" not in code[j]:
                    j -= 1
                assert "lgkmcnt(0)" in code[j], code[max(0, i - 6):i + 1]
            seen += 1
    assert seen == 3
