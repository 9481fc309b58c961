"""Every kernel launch of a call that the runtime rejects ends the call with
PE_EHIP, on every path (tests/launch_driver.c, on the CPU with the runtime's
launch functions replaced)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
def test_every_failed_launch_is_reported(tmp_path):
    import paper_2505_16932_amd as pe
    pe.lib()
    lib = os.path.join(ROOT, "paper_2505_16932_amd", "libpe.so")
    exe = str(tmp_path / "launch_driver")
    subprocess.run(["gcc", "-O1", "-Wall", "-rdynamic", "-o", exe, os.path.join(ROOT, "tests", "launch_driver.c"),
                    "-I", os.path.join(ROOT, "include"), "-ldl"], check=True)
    p = subprocess.run([exe, lib], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    print(p.stdout[-4000:])
    assert p.returncode == 0 and "launch checks: 0 failures" in p.stdout
