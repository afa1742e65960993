"""The kernels that choose whether a node line is read with the non-temporal hint have both loads, as built: the two branches
differ in the hint alone, and a compiler that takes them for the same keeps one, without it.  Disassembly of the built library; no GPU."""
import os
import re
import struct
import subprocess

from paper_2311_17410_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def code_objects(blob):
    """The gfx950 ELF images inside the library (each begins with the ELF magic and names the machine AMDGPU)."""
    at = blob.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:
            shoff, = struct.unpack_from("<Q", blob, at + 40)
            shentsize, shnum = struct.unpack_from("<HH", blob, at + 58)
            yield blob[at:at + shoff + shentsize * shnum]
        at = blob.find(b"\x7fELF", at + 4)


def test_node_lines_are_read_both_ways(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    loads = {}
    for i, image in enumerate(code_objects(open(build.LIB, "rb").read())):
        if b"tns_sample_recent_kernel" not in image and b"tns_sample_kernel" not in image:
            continue
        path = tmp_path / f"{i}.o"
        path.write_bytes(image)
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            wide = re.findall(r"global_load_dwordx4\b.*", part)
            loads[part[:part.index(">")]] = sum(" nt" in w for w in wide), sum(" nt" not in w for w in wide)
    recent = {n: v for n, v in loads.items() if re.search(r"tns_sample_recent_kernelILb0E.*Li[01]EEEv", n)}      # default layout, no small grids
    uniform = {n: v for n, v in loads.items() if re.search(r"tns_sample_kernelILi1E.*Lb0ELi\dEEEv", n)}
    assert len(recent) == 8 and len(uniform) == 12, sorted(loads)
    for name, (hint, plain) in recent.items():
        assert hint >= 8 and plain >= 8, (name, hint, plain)
    for name, (hint, plain) in uniform.items():      # (one of the eight is the same in both branches, which measured faster)
        assert hint >= 7 and plain >= 8, (name, hint, plain)
