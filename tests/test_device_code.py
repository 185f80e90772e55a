"""What the compiler made of the device code, read from the library's own code objects (no GPU needed)."""
import os
import re
import struct
import subprocess

import pytest

import paper_2511_23225_amd as tw
from paper_2511_23225_amd import build as tw_build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """gfx950 ELF files of the library, one a source (uncompressed offload bundles, one behind the other)."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(tw.LIB_PATH):
        tw_build.build_library()
    blob = open(tw.LIB_PATH, "rb").read()
    files, tmp = [], tmp_path_factory.mktemp("code")
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        at = m.end()
        count, = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(count if count < 16 else 0):
            offset, size, length = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name and size:
                files.append(str(tmp / ("%d.elf" % len(files))))
                open(files[-1], "wb").write(blob[m.start() + offset:m.start() + offset + size])
    assert len(files) >= len(tw_build.SOURCES) - 1
    return files


def instructions(code_objects, kernel):
    """{symbol: instruction mnemonics} of the kernels whose name holds `kernel`."""
    found = {}
    for f in code_objects:
        names = [l.split()[-1] for l in subprocess.run([OBJDUMP, "-t", f], capture_output=True, text=True, check=True).stdout.splitlines()
                 if " .text" in l and kernel in l]
        if not names:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", "--disassemble-symbols=" + ",".join(names), f],
                              capture_output=True, text=True, check=True).stdout
        at = None
        for line in text.splitlines():
            m = re.match(r"(?:[0-9a-f]+ )?<(\S+)>:", line)
            if m:
                at = found.setdefault(m.group(1), [])
            elif at is not None and line.strip():
                at.append(line.split()[0])
    return found


# a FLAT access may end out of order and counts in both wait counters: the counted waits for the operand stream allow none
@pytest.mark.parametrize("kernel", ["gemm_nt_defer_kernel", "gemm_nt_defer_mixed_kernel", "gemm_nt_defer_pair_kernel"])
def test_no_flat_access_beside_counted_waits(code_objects, kernel):
    found = instructions(code_objects, kernel)
    assert found and all("s_endpgm" in ops for ops in found.values())
    flat = {name: sum(op.startswith("flat_") for op in ops) for name, ops in found.items()}
    assert not any(flat.values()), flat
