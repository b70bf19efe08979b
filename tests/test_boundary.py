"""CPU-side checks of the C-ABI library: it loads, exports every symbol the
header declares, and rejects bad arguments on the host before touching a GPU.
No compute call is made here."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2208_06874_amd import vp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "vp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(vp_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = _declared_functions()
    assert set(names) == set(vp.EXPORTS)
    L = vp.lib()
    for n in names:
        assert getattr(L, n) is not None


def test_python_binding_has_the_same_names():
    import paper_2208_06874_amd as P
    for n in ("vp_build", "vp_project", "vp_project_full", "vp_project_debug_logits", "vp_workspace_bytes",
              "vp_set_option", "vp_get_info", "vp_get_profile", "vp_destroy", "vp_last_error", "vp_project_union",
              "vp_union_workspace_bytes", "vp_kmeans", "vp_kmeans_workspace_bytes", "vp_active_sets",
              "vp_active_sets_workspace_bytes", "vp_round_to_half", "vp_beam_step", "vp_project_static", "vp_measure_ceilings"):
        assert callable(getattr(P, n))


def _desc(d=64, V=100, K=3, lists=None, k_max=4, flags=0):
    if lists is None:
        lists = [np.arange(0, 40, 2), np.arange(5, 60), np.array([99])]
    off = np.zeros(len(lists) + 1, np.int64)
    np.cumsum([len(x) for x in lists], out=off[1:])
    ids = (np.concatenate(lists) if len(lists) else np.zeros(0)).astype(np.int32)
    desc = vp.make_desc(d, V, K, 0x1000, 0x1000, 0x1000, off, ids, None, 0, k_max, flags)
    return desc, off, ids   # keep the arrays alive


def test_build_bytes_valid_and_monotone():
    L = vp.lib()
    d1, *_k1 = _desc()
    n1 = L.vp_build_bytes(ctypes.byref(d1))
    assert n1 > 0 and n1 % 256 == 0
    d2, *_k2 = _desc(lists=[np.arange(0, 80), np.arange(5, 60), np.array([99])])
    assert L.vp_build_bytes(ctypes.byref(d2)) > n1
    # slab bytes: candidate groups of 16, d padded to 256, 2 bytes each
    info_groups = sum((len(x) + 15) // 16 for x in [np.arange(0, 40, 2), np.arange(5, 60), np.array([99])])
    assert n1 >= info_groups * 16 * 256 * 2 + ((100 + 15) // 16) * 16 * 256 * 2


@pytest.mark.parametrize("kw,status", [
    (dict(d=60), vp.VP_ERR_UNSUPPORTED),          # d % 8 != 0
    (dict(d=0), vp.VP_ERR_UNSUPPORTED),
    (dict(d=8192), vp.VP_ERR_UNSUPPORTED),
    (dict(K=0, lists=[]), vp.VP_ERR_UNSUPPORTED),
    (dict(k_max=0), vp.VP_ERR_UNSUPPORTED),
    (dict(k_max=33), vp.VP_ERR_UNSUPPORTED),
    (dict(flags=2), vp.VP_ERR_INVALID_ARG),            # an unknown flag bit
    (dict(lists=[np.zeros(0, int), np.zeros(0, int), np.zeros(0, int)]), vp.VP_ERR_UNSUPPORTED),   # all sets empty
    (dict(lists=[np.array([3, 2]), np.arange(4), np.arange(3)]), vp.VP_ERR_INVALID_ARG),   # unsorted
    (dict(lists=[np.array([2, 2]), np.arange(4), np.arange(3)]), vp.VP_ERR_INVALID_ARG),   # duplicate
    (dict(lists=[np.array([2, 100]), np.arange(4), np.arange(3)]), vp.VP_ERR_INVALID_ARG),  # id >= V
    (dict(lists=[np.array([-1, 4]), np.arange(4), np.arange(3)]), vp.VP_ERR_INVALID_ARG),  # id < 0
])
def test_build_rejects_bad_descriptions_on_the_host(kw, status):
    L = vp.lib()
    desc, *_keep = _desc(**kw)
    h = ctypes.c_void_p()
    st = L.vp_build(ctypes.byref(desc), None, ctypes.byref(h))
    assert st == status, vp.last_error()
    assert h.value is None
    assert vp.last_error() != ""


def test_build_rejects_null_and_small_arena_before_any_gpu_work():
    L = vp.lib()
    desc, *_keep = _desc()
    h = ctypes.c_void_p()
    assert L.vp_build(ctypes.byref(desc), None, ctypes.byref(h)) == vp.VP_ERR_INVALID_ARG   # null arena
    desc.arena = 0x100000
    desc.arena_bytes = 1024
    assert L.vp_build(ctypes.byref(desc), None, ctypes.byref(h)) == vp.VP_ERR_WORKSPACE
    desc.arena = 0x100010                      # misaligned
    desc.arena_bytes = 1 << 30
    assert L.vp_build(ctypes.byref(desc), None, ctypes.byref(h)) == vp.VP_ERR_INVALID_ARG
    desc.W = None
    desc.arena = 0x100000
    assert L.vp_build(ctypes.byref(desc), None, ctypes.byref(h)) == vp.VP_ERR_INVALID_ARG
    assert L.vp_build(None, None, ctypes.byref(h)) == vp.VP_ERR_INVALID_ARG
    assert L.vp_build_bytes(None) == 0


def test_calls_reject_null_index():
    L = vp.lib()
    assert L.vp_project(None, None, 1, 1, None, None, None, None, 0, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_project_full(None, None, 1, 1, None, None, None, 0, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_project_debug_logits(None, None, 1, 0, None, None, None, 0, None, 0, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_project_union(None, None, 1, 1, None, None, None, None, None, 0, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_union_workspace_bytes(None, 4) == 0
    assert L.vp_workspace_bytes(None, 4) == 0
    assert L.vp_set_option(None, b"rstar", 1) == vp.VP_ERR_INVALID_ARG
    assert L.vp_get_info(None, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_get_profile(None, None, None) == vp.VP_ERR_INVALID_ARG
    L.vp_destroy(None)   # no-op


def test_training_calls_reject_bad_arguments_on_the_host():
    L = vp.lib()
    assert L.vp_kmeans_workspace_bytes(1000, 64, 10) > 0
    assert L.vp_kmeans_workspace_bytes(1000, 60, 10) == 0        # d % 8
    assert L.vp_kmeans_workspace_bytes(0, 64, 10) == 0
    assert L.vp_kmeans_workspace_bytes(1000, 64, 5000) == 0
    assert L.vp_kmeans_workspace_bytes(2000, 64, 10) >= L.vp_kmeans_workspace_bytes(1000, 64, 10)
    assert L.vp_kmeans(None, 10, 64, 4, 1, 0, None, None, None, None, 0, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_kmeans(0x1000, 10, 64, 4, 1, 2, 0x1000, 0x1000, 0x1000, 0x1000, 1 << 30, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_kmeans(0x1000, 10, 64, 4, -1, 0, 0x1000, 0x1000, 0x1000, 0x1000, 1 << 30, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_kmeans(0x1000, 10, 64, 4, 1, 0, 0x1000, 0x1000, 0x1000, 0x1000, 16, None) == vp.VP_ERR_WORKSPACE
    assert "needed" in vp.last_error()
    assert L.vp_kmeans(0x1008, 10, 64, 4, 1, 0, 0x1000, 0x1000, 0x1000, 0x1000, 1 << 30, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_active_sets_workspace_bytes(4, 100) > 0
    assert L.vp_active_sets_workspace_bytes(0, 100) == 0
    tot = ctypes.c_int64(0)
    assert L.vp_active_sets(None, None, 5, 3, 4, 100, None, None, 0, ctypes.byref(tot), None, 0, None) == \
        vp.VP_ERR_INVALID_ARG
    assert L.vp_active_sets(0x1000, 0x1000, 5, 0, 4, 100, 0x1000, 0x1000, 8, ctypes.byref(tot), 0x1000, 1 << 20,
                            None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_active_sets(0x1000, 0x1000, 5, 3, 4, 100, 0x1000, 0x1000, 8, ctypes.byref(tot), 0x1000, 16,
                            None) == vp.VP_ERR_WORKSPACE


def test_beam_step_rejects_bad_arguments_on_the_host():
    L = vp.lib()
    assert L.vp_beam_step(None, None, None, 2, 4, 4, None, None, None, None) == vp.VP_ERR_INVALID_ARG
    assert L.vp_beam_step(0x1000, 0x1000, 0x1000, 2, 128, 32, 0x1000, 0x1000, 0x1000, None) == vp.VP_ERR_UNSUPPORTED
    assert L.vp_beam_step(0x1000, 0x1000, 0x1000, 2, 0, 4, 0x1000, 0x1000, 0x1000, None) == vp.VP_ERR_UNSUPPORTED
    assert L.vp_beam_step(None, None, None, 0, 4, 4, None, None, None, None) == vp.VP_OK   # no sentences: no-op


def test_round_to_half_is_the_library_cast():
    """The host copy of the rounding vp_kmeans applies to a mean: every fp16 value, midpoints, random doubles."""
    pos = np.arange(0, 0x7c00, dtype=np.uint16)
    vals = pos.view(np.float16).astype(np.float64)
    for i in range(len(pos)):
        assert vp.vp_round_to_half(vals[i]) == int(pos[i])
        assert vp.vp_round_to_half(-vals[i]) == int(pos[i]) | 0x8000
    mids = 0.5 * (vals[:-1] + vals[1:])
    r = np.random.default_rng(0)
    v = np.concatenate([mids, -mids, np.nextafter(mids, np.inf), np.nextafter(mids, -np.inf),
                        r.standard_normal(20000), r.standard_normal(5000) * 1e-6, r.standard_normal(5000) * 3e4,
                        r.standard_normal(1000) * 1e-9, r.standard_normal(1000) * 1e6, [65519.9, 65520.0, 1e300, 0.0]])
    with np.errstate(over="ignore"):
        want = v.astype(np.float16).view(np.uint16)
    got = np.array([vp.vp_round_to_half(x) for x in v], np.uint16)
    assert np.array_equal(got, want)


def test_binding_fails_loudly_without_the_library(monkeypatch, tmp_path):
    monkeypatch.setattr(vp, "_lib", None)
    monkeypatch.setattr(vp, "LIB_PATH", str(tmp_path / "libvp.so"))
    with pytest.raises(RuntimeError, match="missing"):
        vp.lib()


def test_product_path_does_not_reach_the_oracle():
    """Nothing under the package may import or name the oracle."""
    pkg = os.path.join(ROOT, "paper_2208_06874_amd")
    for base, _dirs, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(base, f)).read()
                assert "vp_oracle" not in text and "import oracle" not in text and "from oracle" not in text, f


# ------------------------------------------------------------------ host logic: how a projection is cut into work items
@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    import subprocess
    out = tmp_path_factory.mktemp("layout") / "liblayout_shim.so"
    src = os.path.join(ROOT, "tests", "layout_shim.cpp")
    inc = os.path.join(ROOT, "paper_2208_06874_amd", "csrc")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", inc, src, "-o", str(out)], check=True)
    L = ctypes.CDLL(str(out))
    L.shim_tiles_per_wave.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    L.shim_tiles_per_wave_units.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return L


def test_item_sizing_rules(layout):
    """Tiles per wavefront of a plan: at least 1; never more items than asked for; with little work at least
    one item per resident workgroup slot while items stay >= 4 tiles per wavefront; the clustered variant
    never shortens items and, when it lengthens them, the plan fits one round of workgroup slots."""
    r = np.random.default_rng(5)
    for target, min_items in ((8192, 1024), (2048, 1024), (512, 512), (8192, 768)):
        for total in [1, 3, 16, 4095, 4096, 4097, 8192, 15625, 16384, 16385, 60800, 250000, 10 ** 7] + \
                     [int(x) for x in r.integers(1, 400000, 60)]:
            tpw = layout.shim_tiles_per_wave(total, target, min_items)
            assert tpw >= 1
            items = -(-total // (4 * tpw))
            assert items <= max(target, min_items)
            if total >= 16 * max(target, min_items):          # plenty of work: about `target` items
                assert items > max(target, min_items) // 2
            if total <= 16 * min_items and min_items <= target:   # little work: one item per slot, or short items
                assert tpw <= max(1, -(-total // (4 * min_items)))
            for units in (1, 2, 17, 200, 600, 5000):
                t2 = layout.shim_tiles_per_wave_units(total, units, target, min_items)
                assert t2 >= tpw
                if t2 > tpw:
                    ub_before = -(-total // (4 * tpw)) + units
                    assert min_items < ub_before <= 2 * min_items and 2 * units < min_items
                    assert -(-total // (4 * t2)) + units <= min_items + 1


def test_round_filling_item_count_of_the_many_row_kernel(layout):
    """Items of the kernel that runs one workgroup per compute unit: a whole number of candidate ranges per
    row group, at least one; at most eight rounds of the slots (unless there are more row groups than that);
    the plan the planning kernels then make (tiles per wavefront from that count) has no more items than
    asked for; and no choice of fewer rounds would have filled its rounds better."""
    r = np.random.default_rng(9)
    cases = [(1, 256, 15625), (4, 256, 15625), (16, 256, 15625), (86, 256, 15625), (6, 256, 15625), (1024, 256, 15625),
             (3000, 256, 15625), (5, 256, 3), (86, 304, 8000)]
    cases += [(int(a), int(b), int(c)) for a, b, c in zip(r.integers(1, 1500, 200), r.choice([64, 104, 256, 304], 200),
                                                           r.integers(1, 40000, 200))]
    for rgs, slots, vtiles in cases:
        items = layout.shim_rounds_item_count(rgs, slots, vtiles)
        assert items >= rgs and items % rgs == 0
        ranges = items // rgs
        assert ranges <= max(1, vtiles)
        assert items <= 8 * slots or ranges == 1
        # what the planning kernels make of it: ranges of 4 * tpw tiles
        tpw = layout.shim_tiles_per_wave(rgs * vtiles, items, items)
        chunks = -(-vtiles // (4 * tpw))
        assert chunks * rgs <= items
        fill = items / (-(-items // slots) * slots)
        for rounds in range(1, 9):
            rg2 = min(rounds * slots // rgs, vtiles)
            if rg2 < 1:
                continue
            it2 = rgs * rg2
            f2 = it2 / (-(-it2 // slots) * slots)
            assert f2 <= fill + 1e-9 or fill > 0.97, (rgs, slots, vtiles, items, rounds)
            if f2 > 0.97:
                break


def test_item_count_of_many_row_groups(layout):
    """vp_swept_item_count: whole row groups, never more items than the list holds, ranges that every XCD has for itself
    where several XCDs' worth of row groups meet a long vocabulary, and fewer than 16 row groups as ever."""
    r = np.random.default_rng(8)
    for _ in range(400):
        rgs = int(r.integers(1, 1400))
        slots = int(r.choice([1, 7, 64, 104, 256, 304]))
        vtiles = int(np.exp(r.uniform(0, np.log(40000))))
        kt = int(r.choice([8, 16, 24, 32, 40, 48]))
        most = 8 * slots + 8 * rgs * 3
        items = layout.shim_swept_item_count(rgs, slots, vtiles, kt, most)
        rounds = layout.shim_rounds_item_count(rgs, slots, vtiles)
        assert items % rgs == 0 and 1 <= items // rgs <= max(1, vtiles) and items <= max(most, rounds)
        if rgs < 16:
            assert items == rounds
        if slots == 256 and rgs >= 48 and vtiles >= 12000 and kt >= 40:
            assert items // rgs % 8 == 0, (rgs, vtiles, kt, items)


def test_candidate_groups_per_step_of_the_many_row_kernel(layout):
    """Steps of one, two and four groups as items get longer, two where one row group alone reads the bytes only; each line of two
    holds for a range of item lengths (plans cut items in multiples of four groups), not for a single one, and not where
    steps of two leave wavefronts with one step more than others (20 to 28 groups of d_pad = 256 and 512)."""
    for kt in (8, 16, 24, 32, 40, 48):
        for k in (1, 2, 3, 4, 8, 9, 32):
            for shared in (0, 1):
                by_length = {n: layout.shim_step_groups(kt, k, shared, n, 0) for n in range(1, 400)}
                assert set(by_length.values()) <= {1, 2, 4} and by_length[1] == 1 and by_length[399] == 4
                assert all(by_length[n] <= by_length[n + 1] for n in range(1, 399))
                twos = [n for n in range(4, 400, 4) if by_length[n] == 2]
                assert not (shared and twos) and len(twos) != 1, (kt, k, twos)
                if k > 1 and not shared:
                    edges = {8: (12, 16), 16: (12, 16), 24: None, 32: (32, 64), 40: (16, 20), 48: (16, 32)}[kt]
                    assert (twos[0], twos[-1]) == edges if edges else not twos, (kt, k, twos)
                # (items that trade: two steps for every wavefront and the trade between them, d_pad = 256 and 512)
                apart = [n for n in range(1, 400) if layout.shim_step_groups(kt, k, shared, n, 1) != by_length[n]]
                assert apart == ([29, 30, 31, 32] if kt <= 16 and k > 1 and not shared else [])


def test_bounds_and_sets_of_rows_do_not_straddle_lines(layout):
    """The rows' bounds start half a block of 256 bytes behind the workspace's start (sixteen rows in one line, sixty-four in two
    blocks), behind the header; their sets behind them, from a line's start on, inside the first sections' bytes, which are a
    block and 36 bytes a row, rounded up."""
    layout.shim_set_bounds_at.restype = layout.shim_rows_head_bytes.restype = ctypes.c_longlong
    floors, sets = layout.shim_floors_at(), 4 * layout.shim_bound_sets()
    assert floors % 256 == 128
    for N in list(range(1, 3000)) + [4096, 16384, 65535, 65536]:
        at = floors + layout.shim_set_bounds_at(N)
        assert layout.shim_rows_head_bytes(N) == 256 + -(-36 * N // 256) * 256
        assert at % 128 == 0 and at >= floors + 4 * N and at + sets * N <= layout.shim_rows_head_bytes(N), N


def test_which_calls_trade_the_bests_of_sets(layout):
    """Not outside top-4 to top-8, with few rows of an item, below 24 items a row, or in items in steps of one group; several row
    groups up to d_pad = 1024, two from top-6 on; one row group of d_pad = 768 never (14 % slower there)."""
    trades = layout.shim_trades_sets
    V = 10 ** 6
    for kt in (8, 16, 24, 32, 40, 48):
        slots = 64 if kt <= 32 else 48
        for ntiles in range(4, 1000, 4):
            for N in (1, slots // 2, slots * 3 // 4, slots, slots + 1, slots * 7 // 4 - 1, slots * 7 // 4, 2 * slots, 3 * slots, 9 * slots):
                by_k = [k for k in range(1, 33) if trades(kt, k, N, slots, ntiles, V)]
                assert all(4 <= k <= 8 for k in by_k) and by_k == list(range(by_k[0], 9) if by_k else ())
                if N < slots * 3 // 4 or ntiles * 16 * 24 > V or layout.shim_step_groups(kt, 4, N > slots, ntiles, 1) == 1:
                    assert not by_k
                elif N > slots:
                    two = N <= 2 * slots
                    assert by_k == (([] if two else [7, 8]) if kt > 32 else ([] if kt == 32 and N < 112 else [6, 7, 8]) if two else [4, 5, 6, 7, 8])
                elif kt == 24:
                    assert not by_k
    for kt, ntiles, first in ((8, 64, 7), (8, 32, 4), (16, 32, 4), (16, 36, 7), (16, 56, 4), (32, 32, 4), (32, 36, 7), (40, 20, 7), (40, 24, None), (48, 24, None), (48, 28, 4),
                              (48, 48, None), (48, 52, 4)):
        by_k = [k for k in range(1, 33) if trades(kt, k, 48, 64 if kt <= 32 else 48, ntiles, V)]
        assert by_k == ([] if first is None else list(range(first, 9))), (kt, ntiles, by_k)


def test_event_total_of_the_largest_training_call(layout):
    """Every vector that moves is two events.  From 2^30 vectors that move on their total does not fit 31 bits; it must
    still be seen to be more than the n entries of the event list."""
    r = np.random.default_rng(4)
    for n in (1, 1000, 2 ** 30 - 1, 2 ** 30, 2 ** 31 - 1):
        for moved in {0, n // 2, n // 2 + 1, n, int(r.integers(0, n + 1))}:
            total = np.uint32(0)
            with np.errstate(over="ignore"):
                for part in (moved // 3, moved - moved // 3, moved):      # (three clusters' counts)
                    total += np.uint32(part)
            assert layout.shim_sums_begin_anew(ctypes.c_uint32(int(total)), ctypes.c_int64(n)) == (2 * moved > n), (n, moved)


def test_a_double_adds_up_that_many_entries_exactly(layout):
    """Members that came and members that left are bounded by 2^29 each, so together they may pass what a double holds
    in units of 2^-24; the running sums of events are taken over in parts that cannot."""
    n = layout.shim_km_exact_entries()
    largest = int(float(np.finfo(np.float16).max) * 2 ** 24)
    assert n * largest <= 2 ** 53 and 2 * 2 ** 29 * 2 ** 24 > 2 ** 53
    s, units = 0.0, 0
    for i in range(n):
        v = float(np.finfo(np.float16).max) if i else 2.0 ** -24
        s, units = s + v, units + int(v * 2 ** 24)
    assert int(s * 2 ** 24) == units


def test_short_items_bound_of_the_raw_logit_form(layout):
    """The host considers raw logits only for calls of at most 8,192 candidate tiles.  With the default
    sizing (8,192 items asked for, 1,024 workgroup slots) such a plan has at most VP_RAW_TILES tiles per
    wavefront unless its (bucket, row group) units push it just past one round of workgroups, in which case
    the items get longer and the kernel, which checks the plan's figure, keeps its lists."""
    raw = layout.shim_raw_tiles()
    longer = 0
    for total in list(range(1, 8193, 7)) + [8192]:
        for units in (1, 4, 16, 64):
            tpw = layout.shim_tiles_per_wave_units(total, units, 8192, 1024)
            if total + 8 * units <= 8192:
                assert tpw <= raw
            else:
                assert tpw <= raw + 1
                longer += tpw > raw
    assert longer > 0
    assert layout.shim_tiles_per_wave_units(8193 + 4096, 1, 8192, 1024) > raw
    assert layout.shim_partial_floats(8) == 18


def test_workgroup_to_item_maps_take_every_item_once(layout):
    """The two XCD-aware orders in which workgroups take work items: over a grid of the size the host
    launches, every item is taken by exactly one workgroup and no workgroup gets an item outside the list."""
    B = layout.shim_xcd_block_items()
    r = np.random.default_rng(11)
    # clustered plans with heavy buckets: blocks of B consecutive items dealt to the XCDs, rotated starts
    for total in [1, 2, 31, 32, 33, 255, 256, 257, 1000, 2047, 2048, 2049, 8466] + [int(x) for x in r.integers(1, 20000, 40)]:
        grid = total + 8 * B
        got = [layout.shim_item_of_workgroup(wg, total, -B, 0) for wg in range(grid)]
        taken = sorted(x for x in got if x >= 0)
        assert taken == list(range(total)), total
        assert all(x == -1 or 0 <= x < total for x in got)
    # single bucket, several row groups: candidate ranges dealt to the XCDs, a range's row groups together
    for rgs in (2, 3, 4, 16, 64):
        for chunks in (8, 9, 15, 16, 17, 100, 977):
            grid = -(-chunks // 8) * 8 * rgs
            got = [layout.shim_item_of_workgroup(wg, chunks * rgs, rgs, chunks) for wg in range(grid)]
            assert sorted(x for x in got if x >= 0) == list(range(chunks * rgs)), (rgs, chunks)
            # the row groups of one range run on one XCD
            for wg, it in enumerate(got):
                if it >= 0:
                    assert (it // rgs) % 8 == wg % 8
    # no swizzle
    assert [layout.shim_item_of_workgroup(wg, 10, 0, 0) for wg in range(10)] == list(range(10))


def test_even_workgroup_map_takes_every_item_once_and_balances_the_xcds(layout):
    """The map of the one-workgroup-per-compute-unit kernel: over the smallest grid the host launches (the items
    rounded up to eight, or more) every item is taken once, and no XCD gets more than its eighth."""
    r = np.random.default_rng(12)
    for total in [1, 7, 8, 9, 240, 252, 255, 256, 257, 1978, 2048] + [int(x) for x in r.integers(1, 20000, 40)]:
        for grid in (-(-total // 8) * 8, total + 8, -(-total // 8) * 8 + 40):
            got = [layout.shim_item_of_workgroup_even(wg, total) for wg in range(grid)]
            assert sorted(x for x in got if x >= 0) == list(range(total)), (total, grid)
            per_xcd = [sum(1 for wg in range(x, grid, 8) if got[wg] >= 0) for x in range(8)]
            assert max(per_xcd) <= -(-total // 8)


def _fake_index(d=64, k_max=4):
    """An Index object without a library handle: the binding's own checks run before any C call."""
    import torch
    idx = vp.Index.__new__(vp.Index)
    idx.handle = None
    idx.device = torch.device("cuda:0")
    idx.d, idx.V, idx.K, idx.k_max = d, 100, 3, k_max
    idx._ws, idx._uws = {}, {}
    return idx


def test_binding_rejects_host_tensors_and_wrong_shapes_before_any_c_call():
    """A CPU tensor, a strided view or an output of the wrong size would hand the kernels a host pointer or
    a short buffer: the binding raises first (handle is None here, so reaching the C call would fail differently)."""
    import torch
    idx = _fake_index()
    H = torch.zeros((5, 64), dtype=torch.float16)            # host memory
    for call in (lambda: idx.project(H, 2), lambda: idx.project_full(H, 2), lambda: idx.project_union(H, 2),
                 lambda: idx.debug_logits(H),
                 lambda: idx.project_static(H, 2, torch.zeros((5, 2), dtype=torch.int32),
                                            torch.zeros((5, 2), dtype=torch.float32))):
        with pytest.raises(ValueError, match="GPU memory"):
            call()
    with pytest.raises(ValueError, match="hidden must be"):
        idx.project(torch.zeros(64, dtype=torch.float16), 2)
    with pytest.raises(ValueError, match="shape"):
        idx.project(torch.zeros((5, 32), dtype=torch.float16), 2)
    # the checks themselves, on tensors that claim nothing about the GPU
    t = torch.zeros((4, 6), dtype=torch.float32)
    with pytest.raises(ValueError, match="GPU memory"):
        vp._want(t, "t", torch.float32)
    with pytest.raises(TypeError):
        vp._want([1, 2], "t", torch.float32)
    with pytest.raises(ValueError, match="required"):
        vp._want(None, "t", torch.float32)
    assert vp._want(None, "t", torch.float32, optional=True) is None
    with pytest.raises(ValueError, match="contiguous"):
        vp._want(t.t(), "t", torch.float32)
    with pytest.raises(ValueError, match="float16"):
        idx.project(torch.zeros((5, 64), dtype=torch.float32), 2)


def test_build_rejects_bad_tensors_before_any_c_call():
    import torch
    W = torch.zeros((64, 100), dtype=torch.float16)
    b = torch.zeros(100, dtype=torch.float16)
    C = torch.zeros((3, 64), dtype=torch.float16)
    off = np.array([0, 1, 2, 3], np.int64)
    ids = np.array([0, 1, 2], np.int32)
    with pytest.raises(ValueError, match="GPU memory"):
        vp.Index(W, b, C, off, ids)
    with pytest.raises(ValueError, match="W must be"):
        vp.Index(b, b, C, off, ids)
    with pytest.raises(ValueError, match="centroids must be"):
        vp.Index(W, b, torch.zeros((3, 32), dtype=torch.float16), off, ids)
    for fn in (lambda: vp.vp_kmeans(W, C), lambda: vp.vp_active_sets(torch.zeros((4, 2), dtype=torch.int32),
                                                                      torch.zeros(4, dtype=torch.int32), 3, 100),
               lambda: vp.vp_beam_step(torch.zeros((4, 2), dtype=torch.int32), torch.zeros((4, 2)), torch.zeros(4), 2)):
        with pytest.raises(ValueError, match="GPU memory"):
            fn()


def test_build_flag_drops_the_token_major_copy():
    """VP_BUILD_NO_UNION: the arena shrinks by V * d_pad * 2 bytes; other flag bits are refused."""
    L = vp.lib()
    d0, *_k0 = _desc()
    d1, *_k1 = _desc(flags=vp.BUILD_NO_UNION)
    n0, n1 = L.vp_build_bytes(ctypes.byref(d0)), L.vp_build_bytes(ctypes.byref(d1))
    assert n0 - n1 >= 100 * 256 * 2 and n1 > 0
    d2, *_k2 = _desc(flags=2)
    assert L.vp_build_bytes(ctypes.byref(d2)) == 0 and "flag" in vp.last_error()
