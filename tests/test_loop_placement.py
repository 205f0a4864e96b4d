"""Where the main loops of the projection kernels start.  Up to 6 % of a launch depend on the byte of a 64-byte line at which its loop
begins.  The source asks for a byte in front of the loop, but only the compiler knows whether the loop follows at once: this reads
the places out of the library that was built here.  Needs no GPU."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2501_08090_amd import binding as B

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"

# linear_kernel<MT, NF, KS, PRO, WNT, NORM, NW>: byte of a 64-byte line at which the loop over the chunks of K starts (loop_byte in
# linear.hip, which has the figures)
PLACES = {(2, 4, 4, 0, 1, 0, 4): 28, (3, 2, 4, 0, 1, 0, 4): 28, (3, 1, 8, 0, 1, 0, 4): 20, (2, 1, 4, 0, 1, 0, 8): 16,
          (4, 4, 4, 2, 0, 0, 4): 12, (4, 4, 4, 2, 1, 0, 4): 12, (4, 2, 4, 0, 0, 0, 8): 20, (4, 2, 4, 0, 1, 0, 8): 20}
WIDE = [20, 20]  # linear_wide_kernel: its tiles of 512 and of 256 columns


def code_objects(path):
    """the gfx950 code objects of a library's offload bundles"""
    data = open(path, "rb").read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + ln] and size:
                yield data[at + off:at + off + size]
            p += 24 + ln
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def loops(text):
    """{kernel: [byte at which a loop with matrix instructions starts, ...]} of a disassembly, innermost loops only"""
    out = {}
    for name, body in re.findall(r"^[0-9a-f]+ <(\w+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, re.M | re.S):
        ins = [(int(a, 16), t) for t, a in re.findall(r"^\s+(\S.*?)\s*// ([0-9A-F]+):", body, re.M)]
        found = []
        for a, t in ins:
            m = re.match(r"s_c?branch\S*\s+(\d+)", t)
            if not m or int(m.group(1)) < 32768:
                continue
            to = a + 4 + 4 * (int(m.group(1)) - 65536)
            if a - to < 4096 and any(to <= b <= a and "mfma" in u for b, u in ins):  # (further back lies only a kernel's early end)
                found.append(to % 64)
        out[name] = found
    return out


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump here")
def test_main_loops_start_where_they_were_measured(tmp_path):
    B.load()
    got = {}
    for i, code in enumerate(code_objects(B.LIB_PATH)):
        f = tmp_path / ("%d.elf" % i)
        f.write_bytes(code)
        if b"linear_kernel" not in code:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], check=True, capture_output=True, text=True).stdout
        for name, starts in loops(text).items():
            m = re.match(r"_ZN6chiron13linear_kernelILi(\d)ELi(\d)ELi(\d+)ELi(\d)ELb(\d)ELb(\d)ELi(\d)EE", name)
            if m:
                got[tuple(int(v) for v in m.groups())] = starts
            elif "linear_wide_kernel" in name:
                got["wide"] = starts
    assert got["wide"] == WIDE
    for shape, byte in PLACES.items():
        assert got[shape] == [byte], (shape, got[shape])
