"""The exchange of a split cell's chunk grids, in the built library's gfx950 code: the waves
of a workgroup store the grid through the L2, meet at a barrier, and one of them counts the
chunk for the others.  The barrier does not wait for stores in flight, so each wave has to
wait for its own (s_waitcnt vmcnt(0)) between its last such store and the barrier; and the
workgroup that sums the grids has to invalidate before it reads them."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2606_21278_amd as enf

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LIB = os.path.join(os.path.dirname(enf.__file__), "libenufft.so")


def _instructions(lines):
    for l in lines:
        if l.startswith("\t"):
            yield l.split("//")[0].strip()


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler for the built library")
def test_each_wave_waits_for_its_chunk_stores(tmp_path):
    lib = str(tmp_path / "l.so")   # the code objects are extracted beside the file
    shutil.copy(LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=tmp_path)
    kernels = exchanges = 0
    for obj in sorted(tmp_path.glob("l.so.*gfx950")):
        names = subprocess.run([OBJDUMP, "--syms", str(obj)], check=True, capture_output=True, text=True).stdout
        if "fwd_kernel" not in names:
            continue
        dis = subprocess.Popen([OBJDUMP, "-d", "--mcpu=gfx950", str(obj)], stdout=subprocess.PIPE, text=True)
        body, inside = [], False
        for line in dis.stdout:
            if line.startswith("0") and line.rstrip().endswith(">:"):
                if inside and body:
                    n = _check(body)
                    kernels, exchanges = kernels + 1, exchanges + n
                inside, body = "fwd_kernel" in line, []
            elif inside:
                body.append(line)
        assert dis.wait() == 0
        if inside and body:
            kernels, exchanges = kernels + 1, exchanges + _check(body)
    # every build of the forward kernel holds the exchange once
    assert kernels > 0 and exchanges == kernels


def _check(body):
    """The exchanges in one kernel's code, each with its waits."""
    ins = list(_instructions(body))
    stores = [i for i, x in enumerate(ins) if re.match(r"(global|flat)_store_dwordx2 .* sc1$", x)]
    for i in stores:
        b = next(k for k in range(i + 1, len(ins)) if ins[k] == "s_barrier")
        assert any(re.match(r"s_waitcnt vmcnt\(0\)( |$)", x) for x in ins[i + 1:b]), "a store in flight at the barrier"
        # the counter's add, then the barrier behind which the grids are read
        add = next(k for k in range(b + 1, len(ins)) if re.match(r"(global|flat)_atomic_add", ins[k]))
        assert any(x.startswith("buffer_wbl2 sc1") for x in ins[b:add])
        c = next(k for k in range(add + 1, len(ins)) if ins[k] == "s_barrier")
        read = next(k for k in range(c + 1, len(ins)) if re.match(r"(global|flat)_load", ins[k]))
        assert any(x.startswith("buffer_inv sc1") for x in ins[c:read])
    return len(stores)
