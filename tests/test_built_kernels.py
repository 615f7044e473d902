"""What the compiler made of the kernels whose speed and correctness depend on it: read from the code objects inside
the built library (metadata and disassembly, no GPU)."""
import os
import re
import struct
import subprocess

import pytest

import paper_2601_17917_amd as sd

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 ELF images of a library: every offload bundle lists (offset, size, target) of its entries."""
    with open(path, "rb") as f:
        blob = f.read()
    out, at = [], blob.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        (n,) = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, pos)
            target = blob[pos + 24:pos + 24 + tlen].decode()
            pos += 24 + tlen
            if target.endswith("gfx950") and size:
                out.append(blob[at + off:at + off + size])
        at = blob.find(MAGIC, at + len(MAGIC))
    return out


@pytest.fixture(scope="module")
def images(tmp_path_factory):
    if not os.path.exists(sd.LIB_PATH):
        pytest.skip("the library is not built")
    d = tmp_path_factory.mktemp("images")
    paths = []
    for i, image in enumerate(code_objects(sd.LIB_PATH)):
        paths.append(str(d / f"{i}.elf"))
        with open(paths[-1], "wb") as f:
            f.write(image)
    assert paths
    return paths


def tool(name, *args):
    return subprocess.run([os.path.join(LLVM, name), *args], check=True, capture_output=True, text=True).stdout


def disassembly(images, pattern):
    """{kernel name: its instructions} of the kernels whose name matches."""
    out = {}
    for path in images:
        names = [n for n in re.findall(r"\.name:\s+(_Z\S+)", tool("llvm-readelf", "--notes", path)) if re.search(pattern, n)]
        if names:
            text = tool("llvm-objdump", "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(names), path)
            for name, body in re.findall(r"<(_Z\S+)>:\n(.*?)(?=\n\n|\Z)", text, re.S):
                out[name] = [ln.split("//")[0].strip() for ln in body.splitlines() if ln.strip()]
    return out


def test_projection_accumulators_are_read_after_the_wait(images):
    """lm_head_rows_kernel's matrix instructions are inline assembly, so the compiler inserts no wait states behind
    them: s_nop 7 is what separates the last of them from the next instruction that names an accumulator."""
    kernels = disassembly(images, "lm_head_rows_kernel")
    assert len(kernels) == 2
    for name, ins in kernels.items():
        last, waited, loops = None, False, 0
        for i, s in enumerate(ins):
            if s.startswith("v_mfma"):
                last, waited = i, False
            elif s == "s_nop 7" and last == i - 1:
                waited = True
                loops += 1
            elif last is not None and re.search(r"\ba(\d+\b|\[)", s):
                assert waited, f"{name}: {s} {i - last} instructions behind the last matrix instruction, no wait"
        assert loops == 4, name                          # one per chunk size


def test_projection_rows_do_not_spill(images):
    """lm_head_rows_kernel uses every register of a wave; a spill would cost each of its workgroups the stores."""
    seen = 0
    for path in images:
        for entry in tool("llvm-readelf", "--notes", path).split("- .agpr_count")[1:]:
            if "lm_head_rows_kernel" in re.search(r"\.name:\s+(\S+)", entry).group(1):
                seen += 1
                for key in ("private_segment_fixed_size", "vgpr_spill_count", "sgpr_spill_count"):
                    assert int(re.search(r"\.%s:\s+(\d+)" % key, entry).group(1)) == 0, key
    assert seen == 2


def test_attention_waves_lower_their_priority_again(images):
    """The 16-row waves of 128-wide heads raise their priority at every tile's P V; what follows the last tile (merge, epilogue,
    stores) runs at the ordinary one."""
    kernels = {name: [s for s in ins if s.startswith("s_setprio")] for name, ins in disassembly(images, "attn_bf16_kernel").items()}
    raised = {name: prio for name, prio in kernels.items() if prio}
    assert len(raised) == 6 and all("ILi128ELi1E" in name for name in raised)      # every workgroup shape of <128, 1>
    for name, prio in raised.items():
        assert prio[-1] == "s_setprio 0", (name, prio)


def test_fp32_attention_waits_for_its_lds_reads_before_it_overwrites_them(images):
    """The transfers that bring K into LDS are inline assembly and fill the region that the block before was read from: the wait
    in front of them names the LDS reads, whatever waits the compiler places."""
    kernels = disassembly(images, "attention_f32_kernelILi8ELb[01]ELb1E")
    assert len(kernels) == 2
    for name, ins in kernels.items():
        assert any("global_load_lds" in s for s in ins)
        waits = [s for s in ins if s.startswith("s_waitcnt") and "vmcnt(0)" in s and "lgkmcnt(0)" in s]
        assert len(waits) >= 2, name                     # whole blocks, and the last one that is not
