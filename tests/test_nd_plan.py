"""Which kernels the depths of the one-column nested-dissection sweeps get (nd_units in
csrc/coarse_nd.cpp; host code)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("plan") / "nd_plan")
    csrc = os.path.join(ROOT, "paper_1808_04713_amd", "csrc")
    subprocess.run([HIPCC, "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "nd_plan.cpp"), os.path.join(csrc, "setup.cpp"),
                    os.path.join(csrc, "coarse_nd.cpp"), "-o", exe, "-pthread"], check=True, capture_output=True)

    def run(n, l, requested):
        out = subprocess.run([exe, str(n), str(l), str(int(requested))], capture_output=True, text=True, timeout=120)
        assert out.returncode == 0, out.stderr
        return [line.split() for line in out.stdout.splitlines()]
    return run


def test_backward_units_only_where_depths_share_a_launch(plan):
    """A depth of its own runs backward by rows (short sums: 3.7 us against 4.3 in units);
    the small leaves of a requested factor give stages of one launch."""
    fwd, bwd = plan(96, 1, False)
    assert set(bwd) == {"r"} and "u1" in fwd
    fwd, bwd = plan(64, 2, True)
    assert "u1" not in bwd and any(b[0] == "u" for b in bwd) and any(f[0] == "u" and int(f[1:]) > 1 for f in fwd)
