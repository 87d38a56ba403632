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


def _loop_source():
    return open(os.path.join(build.CSRC, "gemm_loop.hpp")).read()


def _clobbers(text):
    return set(re.findall(r'"([a-z0-9]+)"', re.search(r"#define UL_CLOBBERS (?:.*\\\n)*.*", text).group(0)))


def test_every_register_that_the_blocks_write_is_named_to_the_compiler():
    """Scalar registers and m0, and the vector registers of copy offsets; fragments and accumulators are outputs."""
    text = _loop_source()
    written = set(re.findall(r"(?:\\n|\")s_(?!cmp|waitcnt|cbranch|branch|barrier|nop)\w+ (m0|s\d+),", text))
    for first, last in re.findall(r"s_mov_b64 s\[(\d+):(\d+)\],", text):
        written |= {"s%d" % r for r in range(int(first), int(last) + 1)}
    written |= set(re.findall(r'#define UL_ROW_\w "(v\d+)"', text))
    assert {"m0", "s40", "s49"} < written and len(written) == 21, sorted(written)
    assert written <= _clobbers(text), sorted(written - _clobbers(text))


def test_values_kept_over_the_main_loop_are_in_registers_that_it_leaves_alone():
    kept = re.findall(r"UL_KEPT\(\w, ([0-9, ]+)\)", open(os.path.join(build.CSRC, "gemm_tile.hpp")).read())
    kept = [int(r) for eight in kept for r in eight.split(",")]
    assert len(kept) == len(set(kept)) == 32
    assert max(kept) < 128                                    # the fragments' registers
    assert not {"v%d" % r for r in kept} & _clobbers(_loop_source())
