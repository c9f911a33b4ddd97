"""The pages of offspring on the host: the library's own page functions, compiled
for the CPU (see pages_host.hip)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_pages_fit_where_the_offspring_fit(tmp_path):
    exe = str(tmp_path / "pages_host")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17",
                    os.path.join(HERE, "pages_host.hip"), "-o", exe], check=True, capture_output=True, timeout=300)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
