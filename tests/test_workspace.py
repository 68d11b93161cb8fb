"""The intermediate buffers that a batch keeps between calls hold what every network needs that is given
them: tests/sanitize/workspace_driver.cpp over pairs of networks, on the CPU."""
import os
import shutil
import subprocess

import pytest

from tests.test_sanitizers import ENV, FLAGS, ROOT, SAN


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_kept_buffers_fit_every_network_that_takes_them(tmp_path):
    exe, csrc = str(tmp_path / "workspace"), os.path.join(ROOT, "paper_1906_08879_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", *FLAGS, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + csrc, os.path.join(csrc, "workspace.cpp"),
                    os.path.join(SAN, "workspace_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, env=ENV, timeout=300)
    assert r.returncode == 0 and "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, (r.stdout + r.stderr)[-3000:]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_room_of_copies_over_calls_and_captures(tmp_path):
    """Passes of any networks and numbers of steps in any order, replayed captured ones among them, find the tables of their
    copies and stay in their room; a capture changes nothing that the host remembers."""
    exe, csrc = str(tmp_path / "copies"), os.path.join(ROOT, "paper_1906_08879_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", *FLAGS, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + csrc, os.path.join(csrc, "workspace.cpp"),
                    os.path.join(SAN, "copies_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, env=ENV, timeout=300)
    assert r.returncode == 0 and "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, (r.stdout + r.stderr)[-3000:]
