"""Kernels whose last workgroup goes on with what all of them wrote: in the built
code, every wave waits for its own stores and atomics before the barrier behind
which one thread releases them and takes the workgroup's ticket."""

import os
import re
import shutil
import subprocess

import pytest

from paper_1802_05421_amd import _build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KERNELS = ("k_select_pass", "k_select_buffer", "k_degree_stats")


def _functions(tmp_path):
    """Disassembly of the library's device functions, {symbol: [instruction]}."""
    if not os.path.exists(_build.LIB) or not os.path.exists(OBJDUMP):
        pytest.skip("no built library or no llvm-objdump")
    lib = shutil.copy(_build.LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True,
                              capture_output=True, text=True).stdout
        cur = None
        for line in text.splitlines():
            m = re.match(r"^[0-9a-f]+ <(\S+)>:$", line)
            if m:
                cur = out.setdefault(m.group(1), [])
            elif cur is not None and line.strip():
                cur.append(line.split("//")[0].strip())
    return out


def test_waves_wait_for_their_stores_before_the_ticket(tmp_path):
    funcs = {k: v for k, v in _functions(tmp_path).items() if any(n in k for n in KERNELS)}
    assert all(any(n in k for k in funcs) for n in KERNELS)
    for name, ins in funcs.items():
        # (releases that an atomic with its old value returned follows)
        release = [i for i, x in enumerate(ins) if x.startswith("buffer_wbl2")
                   and any(re.match(r"(global|flat)_atomic_add .* sc0", y) for y in ins[i:i + 15])]
        assert len(release) == 1, name
        barrier = max(i for i, x in enumerate(ins[:release[0]]) if x.startswith("s_barrier"))
        wait = [i for i, x in enumerate(ins[:barrier]) if x.startswith("s_waitcnt") and "vmcnt(0)" in x]
        store = [i for i, x in enumerate(ins[:barrier]) if re.match(r"(global|flat|buffer)_(store|atomic)", x)]
        assert wait and store and wait[-1] > store[-1], name
