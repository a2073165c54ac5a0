"""Registers of the float32 search kernels as built (code-object metadata of
libfrbx.so): the work-group forms on grids of up to 128 MBD points hold what
they transform in registers, without spills, three waves per SIMD up to 64
channels (168 registers) and two above."""
import os
import re
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1801_02391_amd", "libfrbx.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf not available")
def test_search_kernels_of_small_mbd_grids_do_not_spill(tmp_path):
    data = open(LIB, "rb").read()
    found = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        n = int.from_bytes(data[m.end():m.end() + 8], "little")
        at = m.end() + 8
        for _ in range(n):   # entries: offset, size, length of the target's name, name
            off, size, ln = (int.from_bytes(data[at + 8 * i:at + 8 * i + 8], "little") for i in range(3))
            target = data[at + 24:at + 24 + ln]
            at += 24 + ln
            if b"gfx950" not in target:
                continue
            elf = tmp_path / "code.o"
            elf.write_bytes(data[m.start() + off:m.start() + off + size])
            notes = subprocess.run([READELF, "--notes", str(elf)], capture_output=True, text=True, check=True).stdout
            for kern in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
                get = lambda k: re.search(rf"\.{k}:\s+(\S+)", kern).group(1)
                found[get("name")] = int(get("vgpr_count")), int(get("vgpr_spill_count"))
    # fringe_kernel<J, M, DUMP, CL, LIST, ROWS, CAND, BLK>
    plain = {}
    for name, regs in found.items():
        m = re.search(r"fringe_kernelILi(\d+)ELi(\d+)ELb0ELb(\d)ELb0ELj0ELb0ELi256E", name)
        if m and int(m.group(2)) <= 128:
            plain[tuple(map(int, m.groups()))] = regs
    assert len(plain) == 6 * 4 * 2, sorted(plain)
    for (J, M, compact), (vgpr, spill) in plain.items():
        assert spill == 0 and vgpr <= (168 if J <= 64 else 256), (J, M, compact, vgpr, spill)
    # with 128 channels and MBD points: the registers of the work-group form's own code, no more
    assert plain[(128, 128, 0)][0] <= 200, plain[(128, 128, 0)]
