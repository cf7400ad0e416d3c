"""How the separable element solves are cut into workgroups (csrc/sep_cut.hpp, host
arithmetic), over the modes, coarse modes, columns and requested widths that a handle
can have."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LDS = 160 * 1024        # a compute unit's shared memory
STATIC = 8 * 16         # of it the kernel's own array, a record per element of a workgroup
COLUMNS = (1, 2, 3, 4, 5, 7, 8, 9, 12, 16, 17, 33, 48, 64)


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("cut") / "element_cut")
    subprocess.run([cxx, "-O1", "-std=c++17", os.path.join(ROOT, "tests", "element_cut.cpp"), "-o", exe], check=True)

    def run(cases):
        """[(n, nr, elements, R, want, padded)] -> [(rc, eg, nchunk, threads, bytes, fits, mixes)]"""
        text = "\n".join(" ".join(str(int(v)) for v in c) for c in cases) + "\n"
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        return [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]
    return run


def test_every_cut_fits_a_compute_unit(cut):
    """n modes per direction, nr <= 4 p of them coarse: the dynamic and the kernel's own
    shared memory together stay within a compute unit's, whatever width is asked for.
    (24 modes, 64 of them coarse, 16 columns: the dynamic part alone fills it.)"""
    cases = [(n, nr, ne, R, want, padded) for n in range(2, 42) for nr in sorted({4, 4 * (n - 1) // 2, 64, 4 * (n - 1)})
             if nr <= 4 * (n - 1) for ne in (4, 1024) for R in COLUMNS for want in (0, 1, 2, 4, 8, 16)
             for padded in (0, 1)]
    assert (24, 64, 1024, 16, 16, 0) in cases
    for c, (rc, eg, nchunk, threads, lds, fits, mixes) in zip(cases, cut(cases)):
        assert lds + STATIC <= LDS, (c, rc, lds)
        assert 1 <= rc <= c[3] and nchunk * rc >= c[3] > (nchunk - 1) * rc, c
        assert 64 <= threads <= 256 and threads % 64 == 0, c


def test_the_autotuner_is_told_which_widths_fit(cut):
    widths = (1, 2, 4, 8, 16)
    for n, nr, most in ((13, 48, 16), (23, 64, 16), (24, 63, 16), (24, 64, 8), (32, 124, 8), (41, 160, 4)):
        fits = [bool(r[5]) for r in cut([(n, nr, 64, 16, w, 0) for w in widths])]
        assert fits == [w <= most for w in widths], (n, nr)



def test_few_workgroups_take_one_round_of_tiles(cut):
    """Where all workgroups are at work at once, four tiles of 16 lines, a wave each, are
    no longer a chain than one: columns that make four tiles stay together, more go by
    single columns up to one per compute unit (of 21 to 32 modes, whose rows four waves
    share, up to two, and two columns up to one), else in the fewest chunks of four
    tiles."""
    resident = {9: 4, 13: 4, 17: 3, 20: 2, 21: 3, 25: 2, 32: 2}
    for ne in (4, 16, 100, 256):
        for n, wgs in resident.items():
            one = 64 // n
            for R in COLUMNS:
                (rc, eg, nchunk, *_), = cut([(n, 16, ne, R, 0, 0)])
                shared = 20 < n <= 32
                if ne * R <= (512 if shared and R > one else 256) and (R > one or shared):
                    assert rc == 1, (n, R, ne)
                elif ne * -(-R // one) < 256 * wgs:
                    assert nchunk == -(-R // one) and n * rc <= 64, (n, R, ne)
                else:
                    assert rc == 1 or ne * nchunk >= 512, (n, R, ne)


def test_cut_columns_of_whole_lines_stay_in_whole_lines(cut):
    """Eight columns fill a cache line.  Of columns that come in whole lines, a chunk
    between one and two lines wide takes one (1,024 elements of 14 modes, 64 columns:
    180 us in chunks of 11, 156 in chunks of 8)."""
    for ne in (256, 1024):
        for n, nr in ((9, 16), (12, 16), (13, 48), (14, 20), (15, 4), (17, 40)):
            for R in (16, 24, 40, 48, 64):
                (rc, eg, nchunk, *_), = cut([(n, nr, ne, R, 0, 0)])
                assert nchunk == 1 or not 8 < rc < 16, (n, R, ne, rc)


def test_the_stage_takes_what_registers_leave_idle(cut):
    """Of the kernels for 25 to 32 modes a compute unit's registers hold two workgroups
    of four waves, so half of its shared memory is each one's (29 modes, 8 columns of
    256 elements: 64 us in chunks of 3, 45 in chunks of 4); of the sampling kernel it
    holds four."""
    for n in range(25, 33):
        for ne in (256, 1024):
            (rc, eg, nchunk, threads, lds, *_), = cut([(n, 16, ne, 8, 0, 0)])
            assert rc >= 4 and 2 * (lds + STATIC) <= LDS, (n, ne)
            (rc, eg, nchunk, threads, lds, *_), = cut([(n, 16, ne, 8, 0, 1)])
            assert 4 * (lds - STATIC) <= LDS, (n, ne)


def test_one_column_of_two_row_tiles_keeps_four_waves_busy(cut):
    for n in range(17, 42):
        for ne in (4, 256, 512, 513, 1024):
            (rc, eg, nchunk, threads, *_), = cut([(n, 16, ne, 1, 0, 0)])
            if eg == 1:
                lines = (n + 15) // 16
                assert threads == (256 if 20 < n <= 32 and ne <= 512 else 64 * lines), (n, ne)


def test_few_workgroups_of_several_kernels_share_a_launch(cut):
    """13 elements of 1 to 32 modes per direction in one launch up to 2,048 workgroups,
    kernel by kernel beyond."""
    mixes = {R: cut([(32, 16, 13, R, 0, 0)])[0][6] for R in (1, 64, 300, 720)}
    assert mixes == {1: 1, 64: 1, 300: 1, 720: 0}
    assert [cut([(17, 16, ne, 1, 0, 0)])[0][6] for ne in (2048, 2049)] == [1, 0]
