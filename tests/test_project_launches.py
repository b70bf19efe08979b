"""Which kernels vp_project launches, read from the launches it makes (no GPU: the program of project_launch_main.cpp stands
in front of the HIP runtime).  A launch that leaves at once costs 3 to 5 us, so the host leaves out what cannot win."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    from paper_2208_06874_amd import vp
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    if not os.path.exists(vp.LIB_PATH):
        pytest.skip("libvp.so is not built")
    exe = tmp_path_factory.mktemp("project") / "project_launch"
    libdir = os.path.dirname(vp.LIB_PATH)
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "project_launch_main.cpp"), "-L", libdir, "-lvp", "-Wl,-rpath," + libdir,
                    "-Wl,--allow-shlib-undefined", "-o", str(exe)], check=True, capture_output=True)

    def run(d, V, K, lo, hi, k, N):
        """The kernels of one call: {name: workgroups}."""
        r = subprocess.run([str(exe)] + [str(v) for v in (d, V, K, lo, hi, k, N)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr
        lines = r.stdout.strip().split("\n")
        assert lines[0] == "%d 0" % N
        return {name: int(grid) for name, grid in (line.rsplit(" ", 1) for line in lines[1:])}

    return run


# sets too short for any of the other forms, whatever the rows do: only Eq. 2, planner, slabs and merge
@pytest.mark.parametrize("d,V,K,lo,hi,k,N", [
    (512, 56750, 361, 38, 77, 1, 1024), (512, 56750, 361, 38, 77, 4, 1421), (1280, 53706, 510, 5, 89, 4, 1201),
    (1024, 154582, 8, 16, 268, 4, 312), (768, 32396, 41, 37, 74, 1, 1927), (256, 127501, 88, 75, 151, 1, 1469),
    (1024, 250000, 1000, 100, 900, 8, 64), (1536, 69552, 10, 1432, 2864, 1, 430), (768, 21002, 599, 76, 1225, 1, 20)])
def test_short_active_sets_launch_the_slabs_only(launches, d, V, K, lo, hi, k, N):
    got = launches(d, V, K, lo, hi, k, N)
    assert not any("project_gemm" in name or "masked" in name for name in got), got
    assert len(got) == 4


# where the planner has a choice both kernels are launched, the many-row one with workgroups for crowded clusters' items on top of
# the masked ones where crowded clusters may pay
@pytest.mark.parametrize("d,V,K,lo,hi,k,N,grouped", [
    (1536, 250000, 500, 2000, 40000, 8, 4096, True), (1024, 250000, 1000, 10000, 20000, 8, 256, False),
    (1024, 128000, 200, 5000, 8000, 8, 64, False), (1024, 142937, 74, 1906, 3812, 8, 2368, True),
    (1024, 250000, 1000, 10000, 20000, 1, 1023, False), (1024, 250000, 1000, 10000, 20000, 1, 1024, True),
    (512, 137200, 6, 3000, 6000, 8, 191, False), (512, 137200, 6, 3000, 6000, 8, 192, True)])
def test_many_row_kernel_is_launched_where_it_may_win(launches, d, V, K, lo, hi, k, N, grouped):
    got = launches(d, V, K, lo, hi, k, N)
    grid = [n for name, n in got.items() if "project_gemm_lds_kernel" in name]
    assert len(grid) == 1 and len(got) == 5, got
    assert (grid[0] >= 512 + 256) == grouped, grid


# the many-row kernel that trades the bests of sets of candidates (project_gemm_lds_kernel's last template argument) only where items
# of the call may trade: not for lists of another length, not with few rows of an item, nor in few ranges of candidates
@pytest.mark.parametrize("d,V,K,lo,hi,k,N,trades", [
    (1024, 128000, 200, 5000, 8000, 8, 64, True), (1024, 250000, 1000, 10000, 20000, 8, 256, True),
    (1024, 250000, 1000, 10000, 20000, 8, 1024, False), (1024, 128000, 200, 5000, 8000, 8, 32, False),
    (1024, 128000, 200, 5000, 8000, 3, 64, False), (1024, 128000, 200, 5000, 8000, 1, 64, False),
    (768, 200000, 100, 9000, 15000, 8, 64, False), (1536, 250000, 500, 2000, 40000, 6, 4096, False), (1024, 100000, 100, 5000, 8000, 4, 192, True)])
def test_kernel_that_trades_is_launched_only_where_items_trade(launches, d, V, K, lo, hi, k, N, trades):
    got = [name for name in launches(d, V, K, lo, hi, k, N) if "project_gemm_lds_kernel" in name]
    assert len(got) == 1
    assert ("ELb%dEEEv" % trades) in got[0], got


@pytest.mark.parametrize("N,K,form", [(64, 1000, None), (65, 40, (1, 1)), (256, 1000, (1, 1)), (256, 1300, (1, 2)), (333, 1990, (1, 4)),
                                      (769, 1990, (2, 4)), (2047, 2000, (2, 8))])
def test_forms_of_the_many_row_eq2_kernel(launches, N, K, form):
    """Row tiles x centroid tiles per wavefront; up to 64 rows the kernel that splits the k-extent."""
    got = list(launches(264, 300, K, 4, 12, 2, N))
    m = [re.search(r"centroid_kernelILi(\d+)ELi(\d+)E", name) for name in got]
    assert [tuple(map(int, x.groups())) for x in m if x] == ([form] if form else [])
    assert any("centroid_small_kernel" in name for name in got) == (form is None)
