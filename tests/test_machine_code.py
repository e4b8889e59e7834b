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


def _registers(text):
    """("v" or "a", number) of every vector register named."""
    regs = set()
    for one, n, many, lo, hi in re.findall(r"\b(?:([va])(\d+)|([va])\[(\d+):(\d+)\])", text):
        regs |= {(one, int(n))} if one else {(many, k) for k in range(int(lo), int(hi) + 1)}
    return regs


def _states(ins):
    """Wait states an instruction stands for."""
    return int(ins.split()[1]) + 1 if ins.startswith("s_nop") else 1


def _since_product(body):
    """Per instruction: the fewest wait states, over all paths, since a matrix product was issued (capped)."""
    cap, index = 64, {at: k for k, (at, _, _) in enumerate(body)}
    since = [None] * len(body)
    work = [(0, cap)]
    while work:
        k, n = work.pop()
        while k < len(body) and (since[k] is None or n < since[k]):
            since[k] = n
            _, ins, target = body[k]
            n = 0 if ins.startswith("v_mfma") else min(cap, n + _states(ins))
            if target is not None:
                work.append((index[target], n))
            if ins.startswith(("s_branch", "s_endpgm")):
                break
            k += 1
    return since


def test_products_finish_before_their_results_are_read(kernels):
    """The block's products are inline assembly: no spill, no accumulator read or stored until the longest
    product's results are there (19 wait states), no operand written by a vector instruction within two wait
    states of a product."""
    seen = 0
    for name, body in kernels.items():
        if "gemm_bf16_kernel" not in name:
            continue
        seen += 1
        since = _since_product(body)
        for k, (at, ins, _) in enumerate(body):
            assert not ins.startswith("scratch_"), f"{name} at {at:x}: {ins}"
            if ins.startswith("v_mfma"):
                near, j = 0, k - 1
                while j >= 0 and near < 2 and not body[j][1].startswith("s_branch"):
                    before = body[j][1]
                    if before.startswith("v_") and not before.startswith("v_mfma"):
                        written = _registers(before.split(",")[0])
                        assert not written & _registers(ins.split(",", 1)[1]), f"{name} at {at:x}: {before}; {ins}"
                    near += _states(before)
                    j -= 1
            elif since[k] is not None and since[k] < 19:
                read = ins if "store" in ins else ins.split(",", 1)[-1]
                assert not any(r == "a" for r, _ in _registers(read)), f"{name} at {at:x}, {since[k]} states: {ins}"
    assert seen == 12
