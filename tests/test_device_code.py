"""CPU-only checks of the compiled kernels: what the hardware's memory order asks of them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_00388_amd import binding as gk


def find_objdump():
    hipcc = shutil.which("hipcc")
    at = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc))), "llvm", "bin") if hipcc else None
    for path in (at, "/opt/rocm/llvm/bin"):
        if path and os.path.exists(os.path.join(path, "llvm-objdump")):
            return os.path.join(path, "llvm-objdump")
    return None


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of every kernel of the library, by name."""
    objdump = find_objdump()
    if objdump is None:
        pytest.skip("no llvm-objdump")
    if not os.path.exists(gk.LIB_PATH):
        from paper_2509_00388_amd import build
        build.build()
    where = tmp_path_factory.mktemp("code")
    lib = shutil.copy(gk.LIB_PATH, where)
    subprocess.run([objdump, "--offloading", lib], cwd=where, check=True, capture_output=True)
    found = {}
    for name in sorted(os.listdir(where)):
        if not name.endswith("gfx950"):
            continue
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", "--no-leading-addr", name], cwd=where, check=True,
                              capture_output=True, text=True).stdout
        body = None
        for line in text.splitlines():
            head = re.match(r"(?:[0-9a-f]+ )?<(_Z\w+)>:", line)
            if head:
                body = found.setdefault(head.group(1), [])
            elif body is not None and line.strip():
                body.append(line.split("//")[0].strip())
    assert found
    return found


def test_stores_are_complete_before_a_workgroup_is_counted(kernels):
    """Where the workgroup that finishes last goes on with what the others wrote, the others count themselves by an
    atomic.  A barrier does not wait for a wave's stores, and a fence of the thread that counts waits for its own
    wave's only: every wave has to wait for its stores in front of the barrier that is in front of the count."""
    counted = {}
    for name, code in kernels.items():
        for at, op in enumerate(code):
            if not (re.match(r"(global|flat)_atomic_(add|inc)\b", op) and "sc0" in op.split()):   # (sc0: the old value is used)
                continue
            barrier = next(i for i in range(at, -1, -1) if code[i].startswith("s_barrier"))
            before = next((code[i] for i in range(barrier, -1, -1)
                           if re.match(r"(global|flat|buffer)_store", code[i]) or re.match(r"s_waitcnt vmcnt\(0\)", code[i])), "")
            counted.setdefault(name, []).append(before)
    for kernel in ("pick_match_kernel", "budget_select_kernel", "redo_decay_kernel"):
        assert any(kernel in name for name in counted), f"{kernel} counts no workgroups"
    bad = {name: ops for name, ops in counted.items() if not all(op.startswith("s_waitcnt") for op in ops)}
    assert not bad, bad
