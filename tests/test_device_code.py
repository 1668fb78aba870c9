"""The built device code: no kernel reaches memory through FLAT instructions.  Every pointer of the kernels is
either global memory or LDS, and the compiler knows which; where it does not (a generic or volatile access
that address-space inference cannot resolve), the access waits for stores it need not wait for, and one that may
be either has faulted on LDS beyond 64 KiB."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_07409_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_flat_access(tmp_path):
    lib = shutil.copy(B.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    objs = sorted(p for p in tmp_path.iterdir() if "gfx950" in p.name)
    assert objs, "no device code in the library"
    kernels, flat = 0, {}
    for o in objs:
        name = "?"
        with subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", o], stdout=subprocess.PIPE, text=True) as p:
            for line in p.stdout:
                m = re.match(r"[0-9a-f]+ <(.+)>:", line)
                if m:
                    name, kernels = m[1], kernels + 1
                elif "\tflat_" in line:
                    flat[name] = flat.get(name, 0) + 1
        assert p.returncode == 0
    assert kernels > 100, kernels
    assert not flat, flat
