"""The stage kernels meet at bare barriers: each wavefront first waits for its own LDS operations,
then signals.  An LDS operation issued between that wait and the barrier could still be under way
when another wavefront reads what it writes, or when the ring slot it reads is refilled.  The source
keeps them apart with compiler fences; here the library built from it is looked at, barrier by
barrier."""
import os
import re
import subprocess

import pytest

from paper_1904_10070_amd import binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def unwaited(listing):
    """(number of barriers, those with an LDS operation since the last wait for all of them)"""
    barriers, late, pending = 0, [], False
    for n, line in enumerate(listing):
        op = line.split("//")[0].split()
        if not op:
            continue
        if op[0].startswith("ds_"):
            pending = True
        elif op[0] == "s_waitcnt" and "lgkmcnt(0)" in line:
            pending = False
        elif op[0] == "s_barrier":
            barriers += 1
            if pending:
                late.append(n)
    return barriers, late


def test_an_unwaited_store_is_found():
    wait, store, barrier = "s_waitcnt vmcnt(5) lgkmcnt(0)", "ds_write_b32 v1, v2", "s_barrier"
    assert unwaited([store, wait, barrier, store, wait, barrier]) == (2, [])
    assert unwaited([store, wait, store, barrier]) == (1, [3])
    assert unwaited([store, "s_waitcnt lgkmcnt(1)", barrier]) == (1, [2])


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_stage_kernels_wait_for_lds_before_every_barrier(tmp_path):
    binding.load_library()
    lib = tmp_path / "libtlb.so"
    lib.symlink_to(binding.LIB_PATH)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, cwd=tmp_path,
                   stdout=subprocess.DEVNULL)
    weno = total = 0
    for code in sorted(tmp_path.glob("*gfx950*")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(code)], check=True,
                              stdout=subprocess.PIPE, text=True).stdout
        for part in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            name, _, body = part.partition(">:")
            if "tlb_stage" not in name:
                continue
            barriers, late = unwaited(body.splitlines())
            assert not late, (name, late[:5])
            total += barriers
            weno += bool(re.search(r"tlb_stage_kernelI[fd]Lb[01]ELi8ELb1E", name))
    assert weno == 8 and total > 500, (weno, total)
