"""The gfx950 code of the built library, disassembled: waits that no run on a GPU
can show to be missing."""
import os
import re
import subprocess

import pytest

from paper_2503_12473_amd import _lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The library's device code objects, unpacked."""
    d = tmp_path_factory.mktemp("code")
    lib = d / "lib.so"
    lib.write_bytes(open(_lib.LIB_PATH, "rb").read())
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=d)
    return sorted(d.glob("lib.so.*gfx950"))


def _kernels(objects, name):
    """Instructions of every kernel `name`, by its symbol."""
    out = {}
    for o in objects:
        syms = subprocess.run([OBJDUMP, "-t", str(o)], check=True, capture_output=True, text=True).stdout
        want = [w for w in re.findall(r"\S+$", syms, re.M) if re.match(rf"_ZN5oecdg\d+{name}\w+$", w)]
        if not want:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(want), str(o)],
                              check=True, capture_output=True, text=True).stdout
        for m in re.finditer(r"^\w+ <(_Z\w+)>:\n((?:.+\n)*)", text, re.M):
            out[m.group(1)] = [re.sub(r"//.*", "", x).split(None, 1) for x in m.group(2).splitlines()]
    return out


def _unwaited_arrivals(ins):
    """Arrivals at an agent-scope counter (global_atomic_add) and those of them whose
    workgroup barrier a wave can pass with a store of its own in flight."""
    arrivals = bad = 0
    for i, x in enumerate(ins):
        if x[0] != "global_atomic_add":
            continue
        arrivals += 1
        j = max(k for k in range(i) if ins[k][0] == "s_barrier")
        for op in reversed(ins[:j]):
            if op[0] == "s_waitcnt" and "vmcnt(0)" in op[1]:
                break
            if op[0].startswith(("global_store", "flat_store")):
                bad += 1
                break
    return arrivals, bad


def test_fold_workgroups_arrive_after_the_stores_of_all_their_waves(code_objects):
    """A workgroup of the fold over many tiles stores its blocks' results from every
    wave; the last to arrive, on whichever XCD, reads them all."""
    kernels = _kernels(code_objects, "k_fold_rows")
    assert len(kernels) == 4
    for name, ins in kernels.items():
        arrivals, bad = _unwaited_arrivals(ins)
        assert arrivals == 2 and bad == 0, name


def test_the_grid_barrier_is_reached_after_the_stores_of_all_waves(code_objects):
    """The persistent launch's grid barrier: every wave's stores (the stage's output and
    statistics, which other workgroups read after it) before the workgroup's arrival."""
    kernels = _kernels(code_objects, "k_persistent")
    assert kernels
    for name, ins in kernels.items():
        arrivals, bad = _unwaited_arrivals(ins)
        assert arrivals >= 1 and bad == 0, name
