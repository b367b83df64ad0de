"""The library's gfx950 machine code as built: per kernel its registers,
spills and occupancy limits (code object metadata) and its instructions."""
import os
import re
import subprocess
import tempfile

from paper_1906_04576_amd import build as b


def _code_object(src, tmp):
    """The device code object of one source: from the built object file, or
    compiled now where nothing is built."""
    obj = os.path.join(b.BUILD, os.path.splitext(src)[0] + ".o")
    if not os.path.exists(obj):
        os.makedirs(b.BUILD, exist_ok=True)
        obj = b._compile(src)
    fat, co = os.path.join(tmp, "fat"), os.path.join(tmp, "co")
    subprocess.run([os.path.join(b.LLVM, "llvm-objcopy"), "--dump-section", f".hip_fatbin={fat}", obj,
                    os.path.join(tmp, "host.o")], check=True, capture_output=True)
    subprocess.run([os.path.join(b.LLVM, "clang-offload-bundler"), "--unbundle", "--type=o",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}", f"--output={co}"],
                   check=True, capture_output=True)
    return co


def kernels(src):
    """{mangled kernel name: {metadata field: int}} of a source."""
    with tempfile.TemporaryDirectory() as tmp:
        co = _code_object(src, tmp)
        text = subprocess.run([os.path.join(b.LLVM, "llvm-readelf"), "--notes", co], check=True, capture_output=True,
                              text=True).stdout
    out = {}
    for part in re.split(r"\n  - (?=\.)", text)[1:]:
        name = re.search(r"\n    \.name:\s+(\S+)", part)
        if name:
            out[name.group(1)] = {k: int(v) for k, v in re.findall(r"\n    \.(\w+):\s+(\d+)(?=\n|$)", part)}
    return out


def waves_per_simd(meta, block=256):
    """Waves of 256-thread blocks that a SIMD holds: 512 vector registers in
    steps of 8, at most 8 waves, and the 160 KB of LDS of a CU's 4 SIMDs."""
    vgprs = (meta["vgpr_count"] + 7) // 8 * 8
    by_regs = min(8, 512 // vgprs)
    lds = meta["group_segment_fixed_size"]
    per_block = block // 64 // 4  # waves of a block on each SIMD
    return min(by_regs, per_block * (160 * 1024 // lds) if lds else 8)


def instructions(src):
    """Mnemonics of a source's device code with their counts."""
    with tempfile.TemporaryDirectory() as tmp:
        co = _code_object(src, tmp)
        text = subprocess.run([os.path.join(b.LLVM, "llvm-objdump"), "-d", "--mcpu=gfx950", "--no-show-raw-insn", co],
                              check=True, capture_output=True, text=True).stdout
    counts = {}
    for m in re.finditer(r"^\s+([a-z]\w+)", text, re.M):
        counts[m.group(1)] = counts.get(m.group(1), 0) + 1
    return counts
