"""The built gfx950 code around inline assembly, whose waits the compiler does
not insert by itself, read from liblsh.so (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2001_04451_amd import lsh

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: [(address, instruction, branch target or None)]} of every device code object."""
    if not os.path.exists(lsh.LIB_PATH):
        pytest.skip("liblsh.so not built (run __graft_entry__.build())")
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    shutil.copy(lsh.LIB_PATH, d / "liblsh.so")
    subprocess.check_call([OBJDUMP, "--offloading", "liblsh.so"], cwd=d, stdout=subprocess.DEVNULL)
    found = {}
    for f in sorted(d.glob("*gfx950")):
        text = subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], text=True)
        start, body = 0, None
        for line in text.splitlines():
            head = re.match(r"([0-9a-f]+) <(\S+)>:", line)
            if head:
                start, body = int(head.group(1), 16), found.setdefault(head.group(2), [])
            elif body is not None and "//" in line:
                ins, note = line.split("//", 1)
                to = re.search(r"<\S+?(?:\+0x([0-9a-f]+))?>", note)
                body.append((int(note.split(":")[0], 16), " ".join(ins.split()),
                             start + int(to.group(1) or "0", 16) if to and ins.split()[0].startswith("s_") else None))
    assert found
    return found


def _copies_to_lds(ins):
    return ins.startswith("global_load_lds") or (ins.startswith("buffer_load") and ins.endswith(" lds"))


def test_lds_copies_wait_for_m0(kernels):
    """A copy to LDS takes its address from m0, and needs a wait state after a scalar write of it."""
    copies = 0
    for name, body in kernels.items():
        for (_, before, _), (at, ins, _) in zip(body, body[1:]):
            if _copies_to_lds(ins):
                copies += 1
                assert not re.match(r"s_\w+ m0,", before), f"{name} at {at:x}: {before}; {ins}"
    assert copies > 100
