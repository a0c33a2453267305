"""The 32x32x16 kernel (k_qmma) waits at its chunk barriers for a counted number of vector
memory operations (s_waitcnt vmcnt), which is right only while a chunk's loads are exactly
the instructions the count assumes: a load the compiler merged, split or dropped would
release the barrier before the chunk's activations are in LDS.  Read from the library
built here, on the CPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_18344_amd import _binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LIB = os.path.join(os.path.dirname(_binding.__file__), "libsubspec.so")


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs the ROCm toolchain")
def test_chunk_barriers_wait_for_the_chunks_loads(tmp_path):
    lib = shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True, timeout=60)
    kernels = {}
    for f in sorted(tmp_path.glob("*gfx950*")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", "--no-leading-addr", str(f)],
                              check=True, capture_output=True, text=True, timeout=120).stdout
        if "k_qmma" not in text:
            continue
        name = None
        for line in text.splitlines():
            m = re.match(r".*<(\w+)>:$", line)
            if m:
                name = m.group(1) if re.match(r"_ZN7subspec4qmma6k_qmmaI", m.group(1)) else None
            elif name:
                kernels.setdefault(name, []).append(line.split())
    assert len(kernels) >= 40, len(kernels)
    for name, code in kernels.items():
        bits, group, mb, nb, xb, waves, teams = (int(v) for v in re.findall(r"Li(\d+)E", name))
        groups = 128 // group  # per chunk
        # two slices of codes and a scale and a zero per group of each column block, the
        # pre-pass sums of x on tiles of more than 64 rows, the copies of x
        chunk = 2 * nb + 2 * groups * nb + (mb > 2) + 32 * mb * teams // (4 * waves)
        what = (bits, group, mb, nb, xb, waves, teams, chunk)
        loads, wait, barriers = 0, None, 0
        for ins in code:
            op = ins[0] if ins else ""
            if op.startswith("buffer_load"):
                loads += 1
            elif op == "s_waitcnt":
                wait = " ".join(ins[1:])
            elif op == "s_barrier":
                if loads:  # a chunk barrier: the loop's start (all but one slot of the ring) or one of its steps
                    assert loads in (chunk, (xb - 1) * chunk), (what, loads)
                    assert re.search(r"vmcnt\(%d\)" % ((xb - 2) * chunk), wait), (what, wait)
                    assert "lgkmcnt(0)" in wait, (what, wait)
                    barriers += 1
                loads, wait = 0, None
        assert barriers >= teams * (xb + 1), (what, barriers)
