"""The resident solver's kernel run on the host under chosen orders of its blocks
(resident_host.cpp): iterates, residuals and iteration counts must not depend on
which block runs ahead or falls behind, whatever the kernel's waits allow."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIP = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP, "hip")),
                                reason="g++ or the HIP headers not available")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("resident_host") / "resident_host")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", "-D__HIP_PLATFORM_AMD__", "-I", HIP,
                        os.path.join(HERE, "resident_host.cpp"), "-o", out, "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def lines(exe, shape, K, R, max_iter, victims, tag=1, tol=1e-12, spin=0, gate=0):
    r = subprocess.run([exe] + [str(v) for v in (*shape, K, R, max_iter, tag, tol, spin, gate, *victims)], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    return r.stdout.splitlines()


@pytest.mark.parametrize("shape,K,R,max_iter,tol", [
    ((150, 8, 4), 8, 4, 40, 1e-12),    # 13 ghost columns, every interval a fold, no refresh
    ((150, 8, 4), 4, 32, 24, 0.3),     # default intervals: checks, and folds after them
    ((150, 8, 4), 16, 2, 48, 1e-12),   # folds between refreshes
    ((223, 8, 4), 3, 1, 12, 1e-12),    # 4 ghost columns, intervals below their depth
    ((224, 8, 4), 4, 2, 24, 1e-12),    # ... at it
    ((223, 8, 4), 5, 1, 20, 1e-12),    # ... above it
    ((300, 8, 4), 4, 32, 16, 0.3),     # three tiles per row
])
def test_order_of_tiles_in_a_row(exe, shape, K, R, max_iter, tol):
    out = lines(exe, shape, K, R, max_iter, range(-1, 2 + (shape[0] > 256)), tol=tol)
    assert len(out) > 2 and len(set(out)) == 1, out


def test_order_of_tiles_in_rows_and_planes(exe):
    out = lines(exe, (30, 17, 9), 4, 32, 12, (-1, 0, 4, 8), tol=0.2)
    assert len(out) == 4 and len(set(out)) == 1, out


@pytest.mark.parametrize("tag", [1, 0x7ffffff0, 0x80000100, 0xffff0000])
def test_tags_of_the_whole_range(exe, tag):
    """Ghost refreshes of a launch late in the tags' range, over flags as a
    cleared buffer holds them."""
    out = lines(exe, (150, 8, 4), 40, 1000, 40, (-1, 0, 1), tag=tag) + lines(exe, (150, 8, 4), 40, 1000, 40, (-1,))
    assert len(out) == 4 and len(set(out)) == 1, out


@pytest.mark.parametrize("shape", [(150, 8, 4), (30, 17, 4)])
@pytest.mark.parametrize("K,R", [(4, 32), (20, 1)])
def test_waits_in_vain(exe, shape, K, R):
    """A wait that gives up after two polls: every block leaves all the same, the
    launch says that it was lost, and what it leaves is finite."""
    for out in lines(exe, shape, K, R, 40, (-1, 0, 1), spin=1):
        assert " lost 1 " in out and out.endswith("finite 1"), out
        assert 0 < int(out.split(" m ")[1].split()[0]) <= 40, out


@pytest.mark.parametrize("shape", [(150, 8, 4), (30, 17, 4)])
def test_roll_call(exe, shape):
    """A launch whose blocks do not all come in time runs whole or not at all,
    whichever block is late."""
    victims = (-1, 0, 1)
    whole = lines(exe, shape, 4, 32, 12, victims)
    early = lines(exe, shape, 4, 32, 12, victims, gate=1)
    assert len(set(whole)) == 1 and " lost 0 " in whole[0] and " m 12 " in whole[0]
    none = {o for o in early if o not in whole}
    assert len(none) == 1, early
    assert " m 0 done 0 lost 2 resid 0 " in none.pop(), early
