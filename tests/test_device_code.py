"""What the hand-written assembly of the lm_head products has to keep and the assembler does not check, read from the
library's own device code (no GPU needed)."""
import os
import re
import struct
import subprocess

import paper_2507_19766_amd as ulorl
from paper_2507_19766_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _device_code(path):
    """The gfx950 code objects embedded in a host library."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        entry = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(MAGIC))[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + name] and size:
                yield data[at + offset:at + offset + size]
            entry += 24 + name
        at = data.find(MAGIC, at + 1)


def test_a_write_of_m0_is_never_followed_at_once_by_a_copy_to_lds(tmp_path):
    """A copy to LDS takes its address from m0, and gfx9 parts need an instruction between a scalar write of m0 and it.  The
    compiler sees to that in its own code, not inside a block of assembly."""
    ulorl.load_library()
    objdump = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin", "llvm-objdump")
    copies, kernel, before, bad = {}, "", "", {}
    for n, code in enumerate(_device_code(ulorl.lib_path())):
        obj = tmp_path / ("%d.co" % n)
        obj.write_bytes(code)
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(obj)], stdout=subprocess.PIPE, text=True, check=True).stdout
        for line in text.splitlines():
            label = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if label:
                kernel, before = label.group(1), ""
            line = line.split("//")[0].strip()
            if re.match(r"buffer_load_dword\S*\s.*\blds$", line):
                copies[kernel] = copies.get(kernel, 0) + 1
                if re.match(r"s_\w+ m0,", before):
                    bad[kernel] = bad.get(kernel, 0) + 1
            before = line
    large = [k for k in copies if "TileLarge" in k]
    assert len(large) == 3 and all(copies[k] > 100 for k in large), copies
    assert not bad, bad
