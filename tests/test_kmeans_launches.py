"""Which membership kernel vp_kmeans takes, read from the launches it makes (no GPU: the program of
kmeans_launch_main.cpp stands in front of the HIP runtime)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MEMBERSHIP = ("kmeans_assign_lds_kernel", "kmeans_assign_gemm_kernel", "centroid_small_kernel", "centroid_kernel")


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    from paper_2208_06874_amd import vp
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    if not os.path.exists(vp.LIB_PATH):
        pytest.skip("libvp.so is not built")
    exe = tmp_path_factory.mktemp("kmeans") / "kmeans_launch"
    libdir = os.path.dirname(vp.LIB_PATH)
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "kmeans_launch_main.cpp"), "-L", libdir, "-lvp", "-Wl,-rpath," + libdir,
                    "-Wl,--allow-shlib-undefined", "-o", str(exe)], check=True, capture_output=True)

    def printed(n, d, K, iters=0, fail_attribute=False):
        r = subprocess.run([str(exe), str(int(fail_attribute)), str(n), str(d), str(K), str(iters)], capture_output=True,
                           text=True, timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout.split("\n")

    def run(n, d, K, iters=0, fail_attribute=False):
        """(status, attribute calls, error left behind, the membership kernel of every pass, which passes keep numbers)"""
        lines = printed(n, d, K, iters, fail_attribute)
        passes = [m for name in lines[3:] for m in MEMBERSHIP if m in name]
        # the counting kernels' RANK argument, as it stands in the mangled names
        kept = [bool(int(b)) for name in lines[3:] for b in re.findall(r"kmeans_assign\w*_kernelI(?:Li\d+E)?Lb([01])E", name)]
        return int(lines[0]), int(lines[1]), int(lines[2]), passes, kept

    run.printed = printed
    return run


@pytest.mark.parametrize("d", [512, 1024, 1536])
def test_lds_size_is_asked_for_once_and_may_be_refused(launches, d):
    """The rows-in-LDS kernel needs its LDS size set.  That is done once a call (for its two forms); if it is refused,
    the split-k kernel serves every pass and the call succeeds with no error left behind."""
    assert launches(8192, d, 1000, iters=3, fail_attribute=True)[:4] == (0, 1, 0, ["kmeans_assign_gemm_kernel"] * 4)
    assert launches(8192, d, 1000, iters=3)[:4] == (0, 2, 0, ["kmeans_assign_lds_kernel"] * 4)


@pytest.mark.parametrize("n,d,K,numbers", [(8192, 1024, 1000, True), (8192, 1024, 200, False), (8192, 256, 256, True),
                                           (8192, 256, 255, False), (3000, 1024, 1000, True), (3000, 1024, 100, False),
                                           (8192, 768, 300, True), (8192, 768, 100, False),
                                           (2 * 256 * 128, 128, 256, True), (2 * 256 * 128 + 1, 128, 256, False)])
def test_members_are_numbered_only_where_the_numbers_are_used(launches, n, d, K, numbers):
    """Passes in front of the means number the members of many clusters, where there is room for the numbers; the last
    pass, and every pass over few clusters, only counts them."""
    assert launches(n, d, K, iters=2)[4] == [numbers, numbers, False]
    assert launches(n, d, K, iters=0)[4] == [False]


@pytest.mark.parametrize("d,n,K,lds", [
    (1024, 4096, 240, False), (1024, 4096, 241, True),                                    # a step for every wavefront
    (1024, 16384, 257, True), (1024, 16385, 257, False), (1024, 16385, 256, True),        # a nearly empty second round
    (1024, 20480, 432, False), (1024, 20481, 432, True), (1000, 16385, 433, True),
    (1024, 49152, 257, True), (1024, 49153, 257, False), (1024, 49153, 304, False), (1024, 49153, 305, True),
    (1024, 57344, 272, False), (1024, 57345, 272, True), (1000, 82000, 272, False), (1024, 98304, 272, True),
    (1536, 12288, 257, True), (1536, 12289, 241, False), (1440, 16384, 480, False),       # one round of the split-k kernel
    (1536, 16384, 481, True), (1536, 16385, 257, True), (1536, 24576, 257, True),
    (1536, 24577, 304, False), (1536, 28160, 272, False), (1536, 28161, 272, True), (1536, 24577, 305, True),
    (1536, 24577, 256, True), (1536, 131072, 272, True),
    (512, 16385, 257, True), (512, 131072, 257, True), (512, 131072, 240, False),
])
def test_membership_kernel_by_size(launches, d, n, K, lds):
    """Both sides of every line of the rule: where the rows-in-LDS kernel measured slower, the other one runs."""
    want = "kmeans_assign_lds_kernel" if lds else "kmeans_assign_gemm_kernel"
    assert launches(n, d, K)[:4] == (0, 2 * int(lds), 0, [want])


@pytest.mark.parametrize("d,n,K,apart", [(1024, 32768, 1000, False), (1024, 32769, 1000, True), (512, 32769, 260, True),
                                         (1536, 24576, 500, False), (1536, 24577, 500, True), (1288, 24577, 500, True),
                                         (1024, 100000, 200, False), (2048, 100000, 500, False)])
def test_passes_are_taken_apart_only_beyond_two_rounds(launches, d, n, K, apart):
    """The companion of the rows-in-LDS kernel is launched in later passes only, and only where two rounds of that kernel
    do not hold all vectors; the split-k kernel takes its passes apart by itself."""
    names = launches.printed(n, d, K, iters=3)[3:]
    assert sum("kmeans_reassign_kernel" in name for name in names) == 3 * int(apart)


@pytest.mark.parametrize("n,d,K,forms", [
    (3000, 1024, 1000, [(1, 8)]), (2000, 264, 1300, [(2, 4)]), (700, 264, 1990, [(1, 2)]), (3900, 264, 1990, [(2, 8)]),
    (66000, 2048, 40, [(1, 1)] * 2), (65536 + 264, 2056, 300, [(2, 4), (1, 4)])])
def test_forms_of_the_decode_time_kernel_in_training(launches, n, d, K, forms):
    """Row tiles x centroid tiles per wavefront, by chunk of 65,536 vectors."""
    names = launches.printed(n, d, K)[3:]
    got = [tuple(map(int, m.groups())) for m in (re.search(r"centroid_kernelILi(\d+)ELi(\d+)E", name) for name in names) if m]
    assert got == forms
