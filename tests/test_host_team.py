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


def test_threads_are_made_as_regions_need_them(build):
    """A mesh of a few classes has regions of a few parts: no more threads than parts,
    and those of earlier regions stay."""
    r = subprocess.run([build("host_team_size")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    most = max(1, min(16, os.cpu_count() or 1))
    size = [int(v) for v in r.stdout.split()]
    assert size[:3] == [1, min(3, most), min(3, most)]
    assert size[3] == size[4] == size[5] <= most and size[3] >= size[1]
