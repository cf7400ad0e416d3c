"""The thread team of the host set-up (csrc/team.hpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def build(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")

    def make(name):
        exe = str(tmp_path_factory.mktemp("team") / name)
        subprocess.run([cxx, "-O1", "-std=c++17", os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe, "-pthread"],
                       check=True)
        return exe
    return make


def test_a_team_without_memory_for_its_threads(build):
    """Whichever allocation of the team fails, the work is done by fewer threads or the
    caller gets std::bad_alloc; threads that run are joined (unjoined, they end the
    process)."""
    r = subprocess.run([build("host_team")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    whole, refused = map(int, r.stdout.split())
    assert whole + refused == 200 and whole > refused
