"""Launch plans of the library's host code (plan_probe.cpp, compiled against the
library's headers and linked with it); no device work."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1804_07250_amd")


@pytest.fixture(scope="module")
def plans():
    """f(requests) -> the probe's answer to each request line."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tempfile.mkdtemp()
    exe = os.path.join(d, "probe")
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                           "-I", os.path.join(PKG, "csrc"), os.path.join(HERE, "plan_probe.cpp"), "-x", "none",
                           os.path.join(PKG, "libtilings.so"), "-Wl,-rpath," + PKG, "-o", exe],
                          stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)

    def ask(requests):
        env = dict(os.environ, LD_LIBRARY_PATH=PKG + os.pathsep + os.environ.get("LD_LIBRARY_PATH", ""))
        r = subprocess.run([exe], input="\n".join(requests) + "\n", capture_output=True, text=True, check=True, env=env)
        out = r.stdout.splitlines()
        assert len(out) == len(requests)
        return out

    yield ask
    shutil.rmtree(d, ignore_errors=True)
