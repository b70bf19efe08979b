"""GPU parity: the HIP library, called through the C ABI, against the CPU oracle
on the same seeded inputs, element by element.  Run with -m gpu on an MI355X."""
import numpy as np
import pytest

from paper_2208_06874_amd import workloads as wl
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


class Built:
    """A workload with its packed index on the GPU."""

    def __init__(self, W, b, C, cand_off, cand_ids, k_max=8, cfg=None):
        torch = _torch()
        from paper_2208_06874_amd import vp
        self.cfg = cfg
        self.W, self.b, self.C = W, b, C
        self.cand_off, self.cand_ids = np.asarray(cand_off, np.int64), np.asarray(cand_ids, np.int32)
        dev = torch.device("cuda:0")
        self.dev = dev
        Wt = torch.from_numpy(W).to(dev)
        bt = torch.from_numpy(b).to(dev)
        Ct = torch.from_numpy(C).to(dev)
        self.index = vp.vp_build(Wt, bt, Ct, self.cand_off, self.cand_ids, k_max=k_max)
        # the tests of this file look at the per-cluster slabs unless they say otherwise: the planner's
        # choice (on by default in the library) is switched on where it is the subject of a test
        self.index.set_option("dispatch", 0)
        torch.cuda.synchronize()
        del Wt, bt, Ct   # the index keeps its own packed copies

    def rows(self, H):
        import torch
        return torch.from_numpy(np.ascontiguousarray(H)).to(self.dev)

    def project(self, H, k, **kw):
        import torch
        ids, logp, g = self.index.project(self.rows(H), k, **kw)
        torch.cuda.synchronize()
        return pu.to_np(ids), pu.to_np(logp), pu.to_np(g)

    def project_full(self, H, k):
        import torch
        ids, logp = self.index.project_full(self.rows(H), k)
        torch.cuda.synchronize()
        return pu.to_np(ids), pu.to_np(logp)

    def project_union(self, H, k):
        import torch
        ids, logp, g, nu = self.index.project_union(self.rows(H), k)
        torch.cuda.synchronize()
        return pu.to_np(ids), pu.to_np(logp), pu.to_np(g), int(nu.item())

    def debug(self, H, full=False):
        import torch
        g, offs, z = self.index.debug_logits(self.rows(H), full=full)
        torch.cuda.synchronize()
        return pu.to_np(g), pu.to_np(offs), pu.to_np(z)


def _from_config(name, **scale):
    _torch()
    cfg = wl.CONFIGS[name]
    if scale:
        cfg = wl.scaled(cfg, **scale)
    W, b, C = wl.make_model(cfg)
    off, ids = wl.make_candidates(cfg, W, b, C, device="cuda:0")
    return Built(W, b, C, off, ids, k_max=8, cfg=cfg)


@pytest.fixture(scope="module")
def tiny():
    return _from_config("tiny")


@pytest.fixture(scope="module")
def mid():
    return _from_config("mid")


@pytest.fixture(scope="module")
def large():
    return _from_config("large")


@pytest.fixture(scope="module")
def skewed():
    return _from_config("skewed")


def _random_lists(r, K, V, lo, hi):
    lists = [np.sort(r.choice(V, size=int(r.integers(lo, hi + 1)), replace=False)) for _ in range(K)]
    off = np.zeros(K + 1, np.int64)
    np.cumsum([len(x) for x in lists], out=off[1:])
    return off, np.concatenate(lists).astype(np.int32)


def _small_model(seed, d, V, K):
    r = np.random.default_rng(seed)
    W = (r.standard_normal((d, V)) / np.sqrt(d)).astype(np.float16)
    b = (r.standard_normal(V) * 0.3).astype(np.float16)
    C = r.standard_normal((K, d)).astype(np.float16)
    return r, W, b, C


def _rows(r, C, N, noise=0.3, clusters=None):
    q = r.integers(0, C.shape[0], N) if clusters is None else np.asarray(clusters)
    return (C[q].astype(np.float32) + noise * r.standard_normal((N, C.shape[1]))).astype(np.float16)


def _full_check(oracle, B, H, k, with_logits=True):
    ids, logp, g = B.project(H, k)
    if with_logits:
        g2, offs, z = B.debug(H)
        assert np.array_equal(g, g2)
    else:
        offs = z = None
    return pu.check_projection(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H, k, ids, logp, g, z, offs)


# ------------------------------------------------------------------ the five workloads
def test_tiny_config(oracle, tiny):
    cfg = tiny.cfg
    H, q = wl.make_rows(cfg, tiny.C)
    st = _full_check(oracle, tiny, H, cfg.k)
    print("tiny", st)
    ids, logp = tiny.project_full(H, cfg.k)
    _, _, zf = tiny.debug(H, full=True)
    print("tiny full", pu.check_full(oracle, tiny.W, tiny.b, H, cfg.k, ids, logp, zf))


def test_mid_config(oracle, mid):
    cfg = mid.cfg
    H, q = wl.make_rows(cfg, mid.C)
    print("mid", _full_check(oracle, mid, H, cfg.k))
    ids, logp = mid.project_full(H[:8], cfg.k)
    print("mid full", pu.check_full(oracle, mid.W, mid.b, H[:8], cfg.k, ids, logp))


def test_large_config(oracle, large):
    cfg = large.cfg
    H, q = wl.make_rows(cfg, large.C)
    print("large", _full_check(oracle, large, H, cfg.k))
    # the full projection at this size: a sample of rows the oracle can afford
    ids, logp = large.project_full(H, cfg.k)
    sample = np.array([0, 17, 101, 255])
    print("large full", pu.check_full(oracle, large.W, large.b, H[sample], cfg.k, ids[sample], logp[sample]))


@pytest.mark.parametrize("N", [1, 4, 16, 64, 256, 1024])
def test_decode_size_sweep(oracle, large, N):
    """Greedy top-1 over the decode-size sweep, rows uniform over clusters."""
    cfg = wl.CONFIGS["sweep"]
    H, q = wl.make_rows(cfg, large.C, N=N, stream=10 + N)
    print("sweep", N, _full_check(oracle, large, H, 1, with_logits=(N <= 64)))


@pytest.mark.parametrize("N,k", [(1, 8), (3, 4), (5, 8), (8, 8), (9, 8)])
def test_few_rows_with_several_candidates_kept(oracle, large, N, k):
    """Few rows, k >= 4: the slab kernel's items are one or two tiles per wavefront and keep raw
    logits instead of per-lane lists (N = 9 is the first size past that bound on this index)."""
    cfg = wl.CONFIGS["sweep"]
    H, q = wl.make_rows(cfg, large.C, N=N, stream=70 + N)
    print("few rows", N, k, _full_check(oracle, large, H, k))


def test_raw_logits_and_lists_agree(tiny, large):
    """The two ways a short item finds its k best (lists built while streaming; raw logits and a selection
    at the end) walk the same total order: same ids, same log-probs."""
    r = np.random.default_rng(71)
    for B, sizes in ((tiny, (1, 7, 16, 40)), (large, (1, 2, 6))):
        for N in sizes:
            H = _rows(r, B.C, N)
            for k in (4, 8):
                got = B.project(H, k)
                B.index.set_option("raw_logits", 0)
                try:
                    ref = B.project(H, k)
                finally:
                    B.index.set_option("raw_logits", 1)
                assert np.array_equal(got[0], ref[0]) and np.array_equal(got[2], ref[2])
                assert np.allclose(got[1], ref[1], rtol=0, atol=1e-5)


def test_skewed_config(oracle, skewed):
    cfg = skewed.cfg
    H, q = wl.make_rows(cfg, skewed.C)
    counts = np.bincount(q, minlength=cfg.K)
    assert counts.max() > 300          # the Zipf head really is a big bucket
    print("skewed", _full_check(oracle, skewed, H, cfg.k, with_logits=False))


# ------------------------------------------------------- the paper's batch-union form
def _union_check(oracle, B, H, k):
    ids, logp, g, nu = B.project_union(H, k)
    return pu.check_union(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H, k, ids, logp, g, nu)


def test_union_worked_example(oracle):
    """Section 2.3: clusters {2,4,6}, {2,8,9}, {1,3} predicted together give the columns {1,2,3,4,6,8,9}."""
    r = np.random.default_rng(0)
    V, d = 10, 64
    W = (r.standard_normal((d, V)) / 3).astype(np.float16)
    b = (r.standard_normal(V) * 0.3).astype(np.float16)
    C = (np.eye(3, d) * 4).astype(np.float16)
    off = np.array([0, 3, 6, 8], np.int64)
    ids = np.array([2, 4, 6, 2, 8, 9, 1, 3], np.int32)
    B = Built(W, b, C, off, ids, k_max=8)
    H = C.copy()
    got_ids, got_logp, g, nu = B.project_union(H, 7)
    assert list(g) == [0, 1, 2] and nu == 7
    for row in got_ids:
        assert sorted(row.tolist()) == [1, 2, 3, 4, 6, 8, 9]
    pu.check_union(oracle, W, b, C, off, ids, H, 7, got_ids, got_logp, g, nu)


def test_union_on_the_workloads(oracle, tiny, mid):
    H, q = wl.make_rows(tiny.cfg, tiny.C)
    print("union tiny", _union_check(oracle, tiny, H, tiny.cfg.k))
    H, q = wl.make_rows(mid.cfg, mid.C, N=8, stream=21)
    print("union mid N=8", _union_check(oracle, mid, H, mid.cfg.k))
    H, q = wl.make_rows(mid.cfg, mid.C, N=40, stream=22)        # the paper's beam 2 x batch 20
    print("union mid N=40", _union_check(oracle, mid, H, mid.cfg.k))


def test_union_equals_per_cluster_form_for_one_cluster(oracle, tiny):
    r = np.random.default_rng(31)
    H = _rows(r, tiny.C, 21, clusters=np.full(21, 5))
    a_ids, a_logp, a_g = tiny.project(H, tiny.cfg.k)
    u_ids, u_logp, u_g, nu = tiny.project_union(H, tiny.cfg.k)
    assert nu == tiny.cand_off[6] - tiny.cand_off[5]
    assert np.array_equal(a_ids, u_ids) and np.array_equal(a_g, u_g)
    assert np.allclose(a_logp, u_logp, rtol=0, atol=1e-5)
    pu.check_union(oracle, tiny.W, tiny.b, tiny.C, tiny.cand_off, tiny.cand_ids, H, tiny.cfg.k, u_ids, u_logp, u_g, nu)


def test_union_ragged_and_large(oracle, large):
    r, W, b, C = _small_model(12, 40, 777, 7)
    off, ids = _random_lists(r, 7, 777, 1, 130)
    B = Built(W, b, C, off, ids, k_max=8)
    for N in (1, 17, 100):
        print("union ragged", N, _union_check(oracle, B, _rows(r, C, N), 3))
    cfg = wl.CONFIGS["sweep"]
    H, q = wl.make_rows(cfg, large.C, N=4, stream=77)
    print("union large N=4", _union_check(oracle, large, H, 8))


# ------------------------------------------------------------------------- edge cases
def test_full_lists_equal_full_projection(oracle):
    r, W, b, C = _small_model(1, 64, 1000, 4)
    off, ids = wl.full_lists(4, 1000)
    B = Built(W, b, C, off, ids, k_max=8)
    H = _rows(r, C, 37)
    a_ids, a_logp, g = B.project(H, 5)
    f_ids, f_logp = B.project_full(H, 5)
    assert np.array_equal(a_ids, f_ids)
    assert np.allclose(a_logp, f_logp, rtol=0, atol=1e-5)
    pu.check_full(oracle, W, b, H, 5, f_ids, f_logp, B.debug(H, full=True)[2])
    pu.check_projection(oracle, W, b, C, off, ids, H, 5, a_ids, a_logp, g)


def test_ragged_shapes(oracle):
    """d not a multiple of the k-tile, list sizes not multiples of 16, N spanning several row groups."""
    r, W, b, C = _small_model(2, 40, 777, 7)
    off, ids = _random_lists(r, 7, 777, 1, 130)
    B = Built(W, b, C, off, ids, k_max=8)
    for N in (1, 15, 16, 17, 100):
        H = _rows(r, C, N)
        print("ragged", N, _full_check(oracle, B, H, 3))


def test_fewer_candidates_than_k(oracle):
    r, W, b, C = _small_model(3, 64, 300, 3)
    lists = [np.array([5]), np.array([1, 7, 299]), np.sort(r.choice(300, 40, replace=False))]
    off = np.array([0, 1, 4, 44], np.int64)
    ids = np.concatenate(lists).astype(np.int32)
    B = Built(W, b, C, off, ids, k_max=8)
    H = _rows(r, C, 9, clusters=[0, 1, 2, 0, 1, 2, 0, 0, 1])
    st = _full_check(oracle, B, H, 8)
    ids_g, logp_g, g = B.project(H, 8)
    one = g == 0
    assert np.all(ids_g[one, 0] == 5) and np.all(logp_g[one, 0] == 0.0) and np.all(ids_g[one, 1:] == -1)
    print("few", st)


def test_all_rows_one_cluster_and_one_row_per_cluster(oracle):
    r, W, b, C = _small_model(4, 128, 5000, 40)
    off, ids = _random_lists(r, 40, 5000, 200, 900)
    B = Built(W, b, C, off, ids, k_max=8)
    H = _rows(r, C, 300, clusters=np.full(300, 11))
    ids_g, logp_g, g = B.project(H, 8)
    assert np.all(g == 11)
    pu.check_projection(oracle, W, b, C, off, ids, H, 8, ids_g, logp_g, g)
    H = _rows(r, C, 40, clusters=np.arange(40))
    ids_g, logp_g, g = B.project(H, 8)
    assert np.array_equal(g, np.arange(40))
    pu.check_projection(oracle, W, b, C, off, ids, H, 8, ids_g, logp_g, g)


def test_duplicate_centroids_and_single_cluster(oracle):
    r, W, b, C = _small_model(5, 64, 400, 6)
    C = np.concatenate([C, C[[2]], C[[0]]], 0)        # clusters 6 and 7 duplicate 2 and 0
    off, ids = _random_lists(r, 8, 400, 20, 60)
    B = Built(W, b, C, off, ids, k_max=4)
    H = _rows(r, C[:6], 24, noise=0.0, clusters=np.arange(24) % 6)    # rows equal to a centroid: exact ties
    ids_g, logp_g, g = B.project(H, 4)
    assert np.array_equal(g, np.arange(24) % 6)       # the lower index wins a tie
    pu.check_projection(oracle, W, b, C, off, ids, H, 4, ids_g, logp_g, g)
    B1 = Built(W, b, C[:1], off[:2], ids[: off[1]], k_max=4)
    H = _rows(r, C, 5)
    ids_g, logp_g, g = B1.project(H, 2)
    assert np.all(g == 0)
    pu.check_projection(oracle, W, b, C[:1], off[:2], ids[: off[1]], H, 2, ids_g, logp_g, g)


def test_equal_logits_tie_goes_to_smaller_token(oracle):
    r, W, b, C = _small_model(6, 64, 200, 2)
    W[:, 150] = W[:, 20] = W[:, 99] = (W[:, 20].astype(np.float32) * 6).astype(np.float16)
    b[150] = b[20] = b[99] = 1.0
    off, ids = wl.full_lists(2, 200)
    B = Built(W, b, C, off, ids, k_max=8)
    H = _rows(r, C, 12)
    a_ids, a_logp, g = B.project(H, 8)
    f_ids, f_logp = B.project_full(H, 8)
    for got in (a_ids, f_ids):
        for row in got:
            row = list(row)
            if 20 in row and 99 in row and 150 in row:
                assert row.index(20) < row.index(99) < row.index(150)
    pu.check_projection(oracle, W, b, C, off, ids, H, 8, a_ids, a_logp, g)
    pu.check_full(oracle, W, b, H, 8, f_ids, f_logp)


def test_empty_batch_and_argument_errors():
    torch = _torch()
    from paper_2208_06874_amd import vp
    r, W, b, C = _small_model(7, 64, 300, 3)
    off, ids = _random_lists(r, 3, 300, 20, 60)
    B = Built(W, b, C, off, ids, k_max=4)
    H0 = torch.empty((0, 64), dtype=torch.float16, device=B.dev)
    ids_g, logp_g, g = B.index.project(H0, 2)
    assert ids_g.shape == (0, 2)
    H = B.rows(_rows(r, C, 4))
    sentinel = torch.full((4, 2), 77, dtype=torch.int32, device=B.dev)
    with pytest.raises(vp.VpError) as e:
        B.index.project(H, 5)                     # k > k_max
    assert e.value.status == vp.VP_ERR_UNSUPPORTED
    with pytest.raises(vp.VpError) as e:
        B.index.project(H, 2, out_ids=sentinel, workspace=torch.empty(256, dtype=torch.uint8, device=B.dev))
    assert e.value.status == vp.VP_ERR_WORKSPACE
    torch.cuda.synchronize()
    assert torch.all(sentinel == 77)              # outputs untouched on error
    info = B.index.info()
    assert info["n_total"] == off[-1] and info["K"] == 3 and info["d_pad"] == 256


def test_largest_topk_and_wide_d(oracle):
    r, W, b, C = _small_model(8, 1536, 3000, 5)
    off, ids = _random_lists(r, 5, 3000, 100, 700)
    B = Built(W, b, C, off, ids, k_max=32)
    H = _rows(r, C, 20)
    ids_g, logp_g, g = B.project(H, 32)
    print("k32", pu.check_projection(oracle, W, b, C, off, ids, H, 32, ids_g, logp_g, g))
    f_ids, f_logp = B.project_full(H, 32)
    pu.check_full(oracle, W, b, H, 32, f_ids, f_logp)


def test_gemv_loop_matches_oracle_and_mfma(oracle, tiny):
    cfg = tiny.cfg
    r = np.random.default_rng(9)
    # buckets of 1..4 rows take the GEMV loop when rstar = 4
    clusters = np.repeat(np.arange(8), [1, 2, 3, 4, 1, 2, 3, 4])
    H = _rows(r, tiny.C, clusters.size, clusters=clusters)
    ref = tiny.project(H, cfg.k)
    tiny.index.set_option("rstar", 4)
    try:
        st = _full_check(oracle, tiny, H, cfg.k)
        got = tiny.project(H, cfg.k)
    finally:
        tiny.index.set_option("rstar", 0)
    print("gemv", st)
    assert np.array_equal(got[2], ref[2])
    assert np.allclose(got[1], ref[1], rtol=0, atol=1e-3)


def test_split_granularity_does_not_change_results(oracle, tiny):
    cfg = tiny.cfg
    H, q = wl.make_rows(cfg, tiny.C, N=40, stream=7)
    base = tiny.project(H, cfg.k)
    for target in (1, 16, 300, 100000):
        tiny.index.set_option("target_items", target)
        tiny.index.set_option("full_target_items", target)
        try:
            got = tiny.project(H, cfg.k)
            f_ids, f_logp = tiny.project_full(H[:5], cfg.k)
        finally:
            tiny.index.set_option("target_items", 8192)
            tiny.index.set_option("full_target_items", 2048)
        assert np.array_equal(got[0], base[0]) and np.array_equal(got[2], base[2])
        assert np.allclose(got[1], base[1], rtol=0, atol=1e-4)
        pu.check_full(oracle, tiny.W, tiny.b, H[:5], cfg.k, f_ids, f_logp)


def test_results_are_deterministic(mid):
    cfg = mid.cfg
    H, q = wl.make_rows(cfg, mid.C, N=200, stream=3)
    a = mid.project(H, cfg.k)
    for _ in range(3):
        c = mid.project(H, cfg.k)
        for x, y in zip(a, c):
            assert np.array_equal(x, y)
    fa = mid.project_full(H[:20], cfg.k)
    fc = mid.project_full(H[:20], cfg.k)
    assert np.array_equal(fa[0], fc[0]) and np.array_equal(fa[1], fc[1])


def test_wide_items_of_the_full_projection(oracle, tiny):
    """From 17 rows on, single-bucket projections use the 64-row kernel; with it switched off, items of 32
    rows (two row tiles per slab tile) for k <= 2, else of 16 rows.  All three must give the same ids."""
    cfg = tiny.cfg
    for N in (24, 75):
        H, q = wl.make_rows(cfg, tiny.C, N=N, stream=9)
        for k in (1, 2):
            default = tiny.project_full(H, k)      # the 64-row kernel
            print("64-row full", N, k, pu.check_full(oracle, tiny.W, tiny.b, H, k, default[0], default[1]))
            tiny.index.set_option("gemm_min_rows", 0)
            try:
                wide = tiny.project_full(H, k)
                print("wide full", N, k, pu.check_full(oracle, tiny.W, tiny.b, H, k, wide[0], wide[1]))
                tiny.index.set_option("wide_items", 0)
                narrow = tiny.project_full(H, k)
                print("narrow full", N, k, pu.check_full(oracle, tiny.W, tiny.b, H, k, narrow[0], narrow[1]))
                ids, logp, g, nu = tiny.project_union(H, 2)
            finally:
                tiny.index.set_option("wide_items", 1)
                tiny.index.set_option("gemm_min_rows", 17)
            for other in (wide, narrow):
                assert np.array_equal(default[0], other[0])
                assert np.allclose(default[1], other[1], rtol=0, atol=1e-4)
            pu.check_union(oracle, tiny.W, tiny.b, tiny.C, tiny.cand_off, tiny.cand_ids, H, 2, ids, logp, g, nu)
    H, q = wl.make_rows(cfg, tiny.C, N=75, stream=9)
    ids, logp, g, nu = tiny.project_union(H, 2)
    pu.check_union(oracle, tiny.W, tiny.b, tiny.C, tiny.cand_off, tiny.cand_ids, H, 2, ids, logp, g, nu)
    _, _, zf = tiny.debug(H[:40], full=True)
    f = oracle.project_full(tiny.W, tiny.b, H[:40], 1, want_all=True)
    assert np.abs(zf.reshape(40, -1) - f["all_z"]).max() < pu.SANITY


def _planner_mode(index, N):
    """White-box: the planner's decision sits in the header at the start of the workspace."""
    import torch
    ws = index.workspace(N)
    torch.cuda.synchronize()
    return int(ws[:64].view(torch.int32)[7].item())


def _overflow(index, N):
    """White-box: the flag that says the plan did not fit its item list (vp.h: VP_WS_OVERFLOW_WORD)."""
    import torch
    ws = index.workspace(N)
    torch.cuda.synchronize()
    return int(ws[:64].view(torch.int32)[2].item())


def test_dispatch_to_the_masked_full_projection(oracle, tiny, mid):
    """With dispatch on, batches that occupy many clusters run the full projection with every row masked
    to its own active set; the results must be those of the per-cluster projection."""
    for B, N, k, want_mode in ((mid, 64, 1, 1), (mid, 200, 1, 1), (mid, 64, 8, 1), (mid, 20, 8, 0), (mid, 2, 8, 0),
                               (tiny, 16, 4, 0), (tiny, 1, 4, 0)):
        cfg = wl.scaled(B.cfg, k=k)
        H, q = wl.make_rows(cfg, B.C, N=N, stream=40 + N)
        base = B.project(H, cfg.k)
        B.index.set_option("dispatch", 1)
        try:
            got = B.project(H, cfg.k)
            mode = _planner_mode(B.index, N)
            st = pu.check_projection(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H, cfg.k, got[0], got[1], got[2])
            # the debug entry keeps the per-cluster layout whatever the option says
            g2, offs, z = B.debug(H)
        finally:
            B.index.set_option("dispatch", 0)
        print("dispatch", cfg.name, N, "mode", mode, st)
        assert mode == want_mode
        assert np.array_equal(got[0], base[0]) and np.array_equal(got[2], base[2])
        assert np.allclose(got[1], base[1], rtol=0, atol=1e-4)
        assert np.array_equal(g2, base[2])
    assert _planner_mode(mid.index, 8) in (0, 1)
    # up to 16 rows: the 16-row form of the masked projection, forced by making the slabs look slow
    cfg = wl.scaled(mid.cfg, k=8)
    H, q = wl.make_rows(cfg, mid.C, N=12, stream=77)
    base = mid.project(H, 8)
    mid.index.set_option("dispatch", 1)
    mid.index.set_option("cost_bw_slab_gbs", 1)
    try:
        got = mid.project(H, 8)
        assert _planner_mode(mid.index, 12) == 1
    finally:
        mid.index.set_option("cost_bw_slab_gbs", 6800)
        mid.index.set_option("dispatch", 0)
    pu.check_projection(oracle, mid.W, mid.b, mid.C, mid.cand_off, mid.cand_ids, H, 8, got[0], got[1], got[2])
    assert np.array_equal(got[0], base[0])


def test_dispatch_cost_model_constants(mid):
    cfg = wl.scaled(mid.cfg, k=1)
    H, q = wl.make_rows(cfg, mid.C, N=64, stream=50)
    mid.index.set_option("dispatch", 1)
    mid.index.set_option("cost_bw_full_gbs", 10)       # make a pass over the whole W look hopeless
    try:
        got = mid.project(H, cfg.k)
        assert _planner_mode(mid.index, 64) == 0
    finally:
        mid.index.set_option("cost_bw_full_gbs", 5100)
        mid.index.set_option("dispatch", 0)
    base = mid.project(H, cfg.k)
    assert np.array_equal(got[0], base[0])


@pytest.mark.parametrize("which,N", [("mid", 48), ("tiny", 7)])
def test_replay_from_a_captured_graph(mid, tiny, which, N):
    """vp_project only enqueues kernels (no allocation, no synchronisation, no memset), so a call can be
    captured into a HIP graph; every replay, with eager work in between, must equal the eager result.  (The
    small case has no planning kernel: the projection workgroups find their own work.)"""
    import torch
    mid = mid if which == "mid" else tiny
    cfg = mid.cfg
    H, q = wl.make_rows(cfg, mid.C, N=N, stream=5)
    H2, _ = wl.make_rows(cfg, mid.C, N=N, stream=6)
    eager = mid.project(H, cfg.k)
    eager2 = mid.project(H2, cfg.k)
    dev = mid.dev
    hbuf = mid.rows(H)
    ids = torch.empty((N, cfg.k), dtype=torch.int32, device=dev)
    logp = torch.empty((N, cfg.k), dtype=torch.float32, device=dev)
    g = torch.empty((N,), dtype=torch.int32, device=dev)
    ws = torch.empty(mid.index.workspace_bytes(N), dtype=torch.uint8, device=dev)
    mid.index.project(hbuf, cfg.k, out_ids=ids, out_logp=logp, out_cluster=g, workspace=ws)   # warm-up
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mid.index.project(hbuf, cfg.k, out_ids=ids, out_logp=logp, out_cluster=g, workspace=ws)
    for rep in range(4):
        src, want = (H, eager) if rep % 2 == 0 else (H2, eager2)
        hbuf.copy_(mid.rows(src))
        ids.fill_(-7)
        logp.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(pu.to_np(ids), want[0]) and np.array_equal(pu.to_np(g), want[2])
        assert np.array_equal(pu.to_np(logp), want[1])
        mid.project(H2 if rep % 2 == 0 else H, cfg.k)     # eager work between replays


def test_union_argument_errors():
    torch = _torch()
    from paper_2208_06874_amd import vp
    r, W, b, C = _small_model(13, 64, 300, 3)
    off, ids = _random_lists(r, 3, 300, 20, 60)
    B = Built(W, b, C, off, ids, k_max=4)
    H = B.rows(_rows(r, C, 4))
    assert B.index.union_workspace_bytes(4) > B.index.workspace_bytes(4)
    with pytest.raises(vp.VpError) as e:
        B.index.project_union(H, 2, workspace=torch.empty(B.index.workspace_bytes(4), dtype=torch.uint8, device=B.dev))
    assert e.value.status == vp.VP_ERR_WORKSPACE
    with pytest.raises(vp.VpError) as e:
        B.index.project_union(H, 9)
    assert e.value.status == vp.VP_ERR_UNSUPPORTED
    out = B.index.project_union(torch.empty((0, 64), dtype=torch.float16, device=B.dev), 2)
    assert out[0].shape == (0, 2)


def test_many_rows_many_clusters(oracle):
    """Row and cluster counts near the top of what the planner handles in one call."""
    r, W, b, C = _small_model(10, 64, 4000, 2500)
    off, ids = _random_lists(r, 2500, 4000, 17, 80)
    B = Built(W, b, C, off, ids, k_max=2)
    H = _rows(r, C, 9000)
    ids_g, logp_g, g = B.project(H, 2)
    print("many", pu.check_projection(oracle, W, b, C, off, ids, H, 2, ids_g, logp_g, g))


def test_limits_of_one_call(oracle):
    """The largest shapes the header allows: N = 65536 rows in one call; d = 4096 with K = 4096 clusters.
    (Not all three at once: the oracle's Eq. 2 alone would be 10^12 double-precision products.)"""
    r, W, b, C = _small_model(12, 64, 1500, 64)
    off, ids = _random_lists(r, 64, 1500, 17, 200)
    B = Built(W, b, C, off, ids, k_max=2)
    H = _rows(r, C, 65536)
    print("limits: 65536 rows", flush=True)
    ids_g, logp_g, g = B.project(H, 2)
    print("limits rows", pu.check_projection(oracle, W, b, C, off, ids, H, 2, ids_g, logp_g, g), flush=True)
    f_ids, f_logp = B.project_full(H[:4096], 2)
    pu.check_full(oracle, W, b, H[:4096], 2, f_ids, f_logp)

    r, W, b, C = _small_model(14, 4096, 1500, 4096)
    off, ids = _random_lists(r, 4096, 1500, 17, 40)
    B = Built(W, b, C, off, ids, k_max=2)
    H = _rows(r, C, 70)
    print("limits: d 4096, K 4096", flush=True)
    ids_g, logp_g, g = B.project(H, 2)
    print("limits d K", pu.check_projection(oracle, W, b, C, off, ids, H, 2, ids_g, logp_g, g), flush=True)
    f_ids, f_logp = B.project_full(H, 2)
    pu.check_full(oracle, W, b, H, 2, f_ids, f_logp)


def test_largest_topk_on_the_many_row_kernel(oracle):
    """top-32 through the 64-row kernel (full projection, union form, masked dispatch) with ragged row counts."""
    r, W, b, C = _small_model(13, 512, 3000, 6)
    off, ids = _random_lists(r, 6, 3000, 200, 900)
    B = Built(W, b, C, off, ids, k_max=32)
    for N in (17, 33, 100, 129):
        H = _rows(r, C, N)
        f_ids, f_logp = B.project_full(H, 32)
        pu.check_full(oracle, W, b, H, 32, f_ids, f_logp)
        u_ids, u_logp, u_g, u_n = B.project_union(H, 32)
        pu.check_union(oracle, W, b, C, off, ids, H, 32, u_ids, u_logp, u_g, u_n)
        B.index.set_option("dispatch", 1)
        B.index.set_option("cost_bw_slab_gbs", 1)      # force the masked projection
        try:
            m_ids, m_logp, m_g = B.project(H, 32)
            assert _planner_mode(B.index, N) == 1
        finally:
            B.index.set_option("cost_bw_slab_gbs", 6800)
            B.index.set_option("dispatch", 0)
        pu.check_projection(oracle, W, b, C, off, ids, H, 32, m_ids, m_logp, m_g)


def test_shared_workspace_and_side_stream(oracle, mid):
    """One big workspace reused by calls of different sizes and kinds, all on a stream of their own, must give
    what fresh workspaces on the default stream give: nothing may survive in the workspace from call to call,
    and no kernel may run on another stream than the caller's."""
    import torch
    cfg = mid.cfg
    dev = mid.dev
    big = torch.empty(mid.index.union_workspace_bytes(1024), dtype=torch.uint8, device=dev)
    side = torch.cuda.Stream(device=dev)             # default priority
    batches = {N: wl.make_rows(cfg, mid.C, N=N, stream=300 + N)[0] for N in (1024, 5, 70, 33, 17)}
    want = {}
    for N, H in batches.items():
        want[N] = (mid.project(H, 8), mid.project_full(H, 2), mid.project_union(H, 8))
    mid.index.set_option("dispatch", 1)
    try:
        for N, H in batches.items():
            want[N] += (mid.project(H, 8),)
        torch.cuda.synchronize()
        big.fill_(0xA5)                               # stale garbage to start from
        got = {}
        with torch.cuda.stream(side):
            for N, H in batches.items():
                h = mid.rows(H)
                a = mid.index.project(h, 8, workspace=big)
                mid.index.set_option("dispatch", 0)
                b = mid.index.project(h, 8, workspace=big)
                c = mid.index.project_full(h, 2, workspace=big)
                d = mid.index.project_union(h, 8, workspace=big)
                mid.index.set_option("dispatch", 1)
                got[N] = (b, c, d, a)
        side.synchronize()
    finally:
        mid.index.set_option("dispatch", 0)
    for N in batches:
        for kind, (g, w) in enumerate(zip(got[N], want[N])):
            assert np.array_equal(pu.to_np(g[0]), w[0]), (N, kind)
            assert np.array_equal(pu.to_np(g[1]), w[1]), (N, kind)


@pytest.mark.parametrize("d,gemm_lds", [(1536, 0), (2048, 1), (1536, 1)])
def test_many_row_kernels_beyond_d_1024(oracle, d, gemm_lds):
    """Beyond d = 1024: the split-k kernel with eight wavefronts (d = 2048, or d = 1536 with the other kernel
    switched off), and at d = 1536 the kernel with the rows in LDS, 48 rows per item (ragged row counts around
    multiples of 48, top-1 to top-32)."""
    r, W, b, C = _small_model(16 + d, d, 1200, 4)
    off, ids = _random_lists(r, 4, 1200, 100, 500)
    B = Built(W, b, C, off, ids, k_max=32)
    B.index.set_option("gemm_lds", gemm_lds)
    cases = ((40, 3), (150, 8)) if not (d == 1536 and gemm_lds) else ((17, 1), (48, 8), (49, 32), (97, 2), (150, 8))
    for N, k in cases:
        H = _rows(r, C, N)
        f_ids, f_logp = B.project_full(H, k)
        print("eight slices full", d, N, pu.check_full(oracle, W, b, H, k, f_ids, f_logp))
        u_ids, u_logp, u_g, u_n = B.project_union(H, k)
        pu.check_union(oracle, W, b, C, off, ids, H, k, u_ids, u_logp, u_g, u_n)
        B.index.set_option("dispatch", 1)
        B.index.set_option("cost_bw_slab_gbs", 1)      # force the masked projection
        try:
            m_ids, m_logp, m_g = B.project(H, k)
            assert _planner_mode(B.index, N) == 1
        finally:
            B.index.set_option("cost_bw_slab_gbs", 6800)
            B.index.set_option("dispatch", 0)
        pu.check_projection(oracle, W, b, C, off, ids, H, k, m_ids, m_logp, m_g)


@pytest.mark.parametrize("d", [760, 768, 1032, 1280])
def test_many_row_kernel_at_d_pad_768_and_1280(oracle, d):
    """The rows-in-LDS kernel at d_pad 768 (64 rows per item) and 1280 (48): row counts around its items, a width
    that fills the last k-tiles with zeros, top-1 (kept in registers) to top-32, plain, union and masked."""
    r, W, b, C = _small_model(30 + d, d, 1200, 4)
    off, ids = _random_lists(r, 4, 1200, 100, 500)
    B = Built(W, b, C, off, ids, k_max=32)
    per = 64 if d <= 768 else 48
    for N, k in ((17, 1), (per, 8), (per + 1, 32), (2 * per + 1, 2)):
        H = _rows(r, C, N)
        f_ids, f_logp = B.project_full(H, k)
        pu.check_full(oracle, W, b, H, k, f_ids, f_logp)
        u_ids, u_logp, u_g, u_n = B.project_union(H, k)
        pu.check_union(oracle, W, b, C, off, ids, H, k, u_ids, u_logp, u_g, u_n)
        B.index.set_option("dispatch", 1)
        B.index.set_option("cost_bw_slab_gbs", 1)      # force the masked projection
        try:
            m_ids, m_logp, m_g = B.project(H, k)
            assert _planner_mode(B.index, N) == 1
        finally:
            B.index.set_option("cost_bw_slab_gbs", 6800)
            B.index.set_option("dispatch", 0)
        pu.check_projection(oracle, W, b, C, off, ids, H, k, m_ids, m_logp, m_g)


@pytest.mark.parametrize("d,k,N", [(256, 8, 700), (512, 1, 1009), (1000, 8, 640), (1280, 32, 701), (1536, 2, 661)])
def test_some_clusters_masked_and_some_on_slabs(oracle, d, k, N):
    """Crowded and nearly empty clusters in one batch: the planner masks the full projection for the rows of some clusters
    and keeps the slabs of the others (plan mode 2).  Same results as the slabs alone and as the oracle, run twice to
    the bit, with an empty active set among the clusters, top-1 to top-32, 64 and 48 rows per masked item."""
    V, K = 3000, 40
    r, W, b, C = _small_model(60 + d + k, d, V, K)
    lists = [np.sort(r.choice(V, size=n, replace=False)) for n in np.r_[0, r.integers(1, 20, 3), r.integers(200, 1500, K - 4)]]
    off = np.zeros(K + 1, np.int64)
    np.cumsum([len(x) for x in lists], out=off[1:])
    ids = np.concatenate(lists).astype(np.int32)
    B = Built(W, b, C, off, ids, k_max=32)
    p = np.arange(1, K + 1) ** -1.3
    q = r.choice(r.permutation(K), size=N, p=p / p.sum())
    q[:K] = np.arange(K)
    H = _rows(r, C, N, clusters=q)
    base = B.project(H, k)
    B.index.set_option("dispatch", 1)
    # rates that make a slab's price its bytes alone, however many rows share it, and the times long beside the
    # planner's fixed ones
    rates = {"cost_row_slab_ns": (0, 60), "cost_bw_l2_gbs": (1000000, 17000), "cost_bw_full_gbs": (1000000, 5100),
             "cost_bw_slab_gbs": (7, 6800), "cost_bw_gemm_gbs": (14, 14000)}
    try:
        for name, (v, _) in rates.items():
            B.index.set_option(name, v)
        got = B.project(H, k)
        assert _planner_mode(B.index, N) == 2
        assert _overflow(B.index, N) == 0
        again = B.project(H, k)
    finally:
        for name, (_, v) in rates.items():
            B.index.set_option(name, v)
        B.index.set_option("dispatch", 0)
    for x, y in zip(got, again):
        assert np.array_equal(x, y)
    assert np.array_equal(got[0], base[0]) and np.array_equal(got[2], base[2])
    assert np.allclose(got[1], base[1], rtol=0, atol=1e-4)
    pu.check_projection(oracle, W, b, C, off, ids, H, k, got[0], got[1], got[2])


@pytest.mark.parametrize("d,k,N,K", [(256, 1, 200, 3), (512, 8, 1100, 40), (768, 4, 65, 2), (1000, 32, 640, 12),
                                     (1280, 2, 1031, 60), (1536, 8, 500, 9)])
def test_crowded_clusters_on_the_many_row_kernel(oracle, d, k, N, K):
    """Clusters of 33 rows and more go to the many-row kernel with their own slabs, clusters of a few rows stay on the slab
    kernel or are masked, in one plan.  Row counts off every multiple, short and empty lists, top-1 to top-32."""
    V = 12000
    r, W, b, C = _small_model(90 + d + k, d, V, K)
    sizes = np.r_[r.integers(300, 2000, K - 1), 7 if K > 2 else 500]
    if K > 5:
        sizes[2] = 0
    lists = [np.sort(r.choice(V, size=n, replace=False)) for n in sizes]
    off = np.zeros(K + 1, np.int64)
    np.cumsum([len(x) for x in lists], out=off[1:])
    ids = np.concatenate(lists).astype(np.int32)
    B = Built(W, b, C, off, ids, k_max=32)
    p = np.arange(1, K + 1) ** -1.0
    q = r.choice(r.permutation(K), size=N, p=p / p.sum())
    q[:K] = np.arange(K)
    H = _rows(r, C, N, clusters=q)
    base = B.project(H, k)
    B.index.set_option("dispatch", 1)
    # the usual rates, all a thousandth: times that are long beside the planner's fixed ones
    rates = {"cost_row_slab_ns": (0, 60), "cost_bw_slab_gbs": (7, 6800), "cost_bw_l2_gbs": (17, 17000),
             "cost_bw_full_gbs": (5, 5100), "cost_bw_gemm_gbs": (14, 14000)}
    try:
        for name, (v, _) in rates.items():
            B.index.set_option(name, v)
        got = B.project(H, k)
        assert _planner_mode(B.index, N) == 2 and _overflow(B.index, N) == 0
        ws = B.index.workspace(N)
        assert int(ws[:64].view(_torch().int32)[12].item()) > 0      # (items of crowded clusters)
        again = B.project(H, k)
    finally:
        for name, (_, v) in rates.items():
            B.index.set_option(name, v)
        B.index.set_option("dispatch", 0)
    for x, y in zip(got, again):
        assert np.array_equal(x, y)
    assert np.array_equal(got[0], base[0]) and np.array_equal(got[2], base[2])
    assert np.allclose(got[1], base[1], rtol=0, atol=1e-4, equal_nan=True)
    pu.check_projection(oracle, W, b, C, off, ids, H, k, got[0], got[1], got[2])


@pytest.mark.parametrize("d,N", [(256, 64), (512, 128), (768, 61), (1024, 64), (1024, 128), (1280, 48), (1536, 96)])
def test_items_at_the_lines_between_the_step_widths(oracle, d, N):
    """The rows-in-LDS kernel walks short items one candidate group a step, longer ones four: items of 8 to 32 groups on both
    sides of every line (by k-extent, top-1 or lists, one row group or two), the last one short and ragged.  Eight items,
    whole rounds of the option's count."""
    per = 64 if d <= 1024 else 48
    rgs = (N + per - 1) // per
    for groups in (8, 12, 16, 28, 32):
        V = 16 * groups * (8 // rgs) - 21
        r, W, b, C = _small_model(40 + d + groups, d, V, 2)
        off, ids = _random_lists(r, 2, V, 20, 60)
        B = Built(W, b, C, off, ids, k_max=8)
        B.index.set_option("gemm_lds_items", 8)
        H = _rows(r, C, N)
        for k in (1, 2, 3, 8):
            f_ids, f_logp = B.project_full(H, k)
            ws = B.index.workspace(N)
            assert ws[:64].view(_torch().int32)[1].item() * 4 == groups, "the plan's items are of another size"
            pu.check_full(oracle, W, b, H, k, f_ids, f_logp)


def test_all_three_forms_in_one_plan_at_the_usual_rates(oracle):
    """At the rates that users run the planner itself masks some clusters, sends crowded ones to the many-row kernel and keeps
    the others on the slab kernel: same results as the slabs alone and as the oracle, twice to the bit."""
    d, V, K, N, k = 512, 60000, 300, 1500, 4
    r, W, b, C = _small_model(17, d, V, K)
    sizes = np.exp(r.uniform(np.log(50), np.log(15000), K)).astype(np.int64)
    off = np.zeros(K + 1, np.int64)
    np.cumsum(sizes, out=off[1:])
    ids = np.concatenate([np.sort(r.choice(V, size=n, replace=False)) for n in sizes]).astype(np.int32)
    B = Built(W, b, C, off, ids)
    p = np.arange(1, K + 1) ** -1.3
    q = r.choice(r.permutation(K), size=N, p=p / p.sum())
    q[:K] = np.arange(K)
    H = _rows(r, C, N, clusters=q)
    base = B.project(H, k)
    B.index.set_option("dispatch", 1)
    got = B.project(H, k)
    assert _planner_mode(B.index, N) == 2 and _overflow(B.index, N) == 0
    hdr = B.index.workspace(N)[:64].view(_torch().int32).tolist()
    assert hdr[0] > 0 and hdr[8] > 0 and hdr[12] > 0, hdr      # (items of slabs, masked, of crowded clusters)
    again = B.project(H, k)
    for x, y in zip(got, again):
        assert np.array_equal(x, y)
    assert np.array_equal(got[0], base[0]) and np.array_equal(got[2], base[2])
    assert np.allclose(got[1], base[1], rtol=0, atol=1e-4)
    pu.check_projection(oracle, W, b, C, off, ids, H, k, got[0], got[1], got[2])


def test_empty_active_sets(oracle):
    """A cluster whose active set is empty (a cluster that lost its members in training): rows that fall into
    it get ids -1 and log-probs -inf in every form of the projection; the other rows are untouched."""
    r, W, b, C = _small_model(15, 128, 900, 6)
    lists = [np.sort(r.choice(900, size=n, replace=False)) for n in (40, 0, 170, 0, 33, 5)]
    off = np.zeros(7, np.int64)
    np.cumsum([len(x) for x in lists], out=off[1:])
    ids = np.concatenate(lists).astype(np.int32)
    B = Built(W, b, C, off, ids, k_max=4)
    for N in (9, 70):
        H = _rows(r, C, N, clusters=np.arange(N) % 6)
        ids_g, logp_g, g = B.project(H, 4)
        st = pu.check_projection(oracle, W, b, C, off, ids, H, 4, ids_g, logp_g, g)
        hit = np.isin(g, (1, 3))
        assert hit.any() and np.all(ids_g[hit] == -1) and np.all(np.isneginf(logp_g[hit]))
        assert np.all(ids_g[~hit][:, 0] >= 0)
        g2, offs, z = B.debug(H)
        assert np.array_equal(offs, oracle.project(W, b, C, off, ids, H, 4, forced_g=g, want_all=True)["all_off"])
        u_ids, u_logp, u_g, u_n = B.project_union(H, 4)
        pu.check_union(oracle, W, b, C, off, ids, H, 4, u_ids, u_logp, u_g, u_n)
        B.index.set_option("dispatch", 1)
        B.index.set_option("cost_bw_slab_gbs", 1)      # force the masked projection
        try:
            m_ids, m_logp, m_g = B.project(H, 4)
            assert _planner_mode(B.index, N) == 1
        finally:
            B.index.set_option("cost_bw_slab_gbs", 6800)
            B.index.set_option("dispatch", 0)
        assert np.array_equal(m_ids, ids_g) and np.allclose(m_logp, logp_g, rtol=0, atol=1e-4, equal_nan=True)
        print("empty sets", N, st)
    # a batch that only meets empty clusters: the union is empty
    H = _rows(r, C, 5, clusters=np.array([1, 3, 1, 1, 3]), noise=0.01)
    u_ids, u_logp, u_g, u_n = B.project_union(H, 4)
    assert u_n == 0 and np.all(u_ids == -1) and np.all(np.isneginf(u_logp))


def test_non_finite_rows_stay_in_their_lane(tiny):
    """A row with NaN or infinite entries gets meaningless values, but every index stays in range, the call
    completes, and the other rows of the batch are exactly what they are without it."""
    cfg = tiny.cfg
    H, q = wl.make_rows(cfg, tiny.C, N=40, stream=91)
    bad = H.copy()
    bad[3, 5] = np.float16(np.nan)
    bad[17, :] = np.float16(np.inf)
    bad[29, 0] = np.float16(-np.inf)
    good_rows = np.setdiff1d(np.arange(40), [3, 17, 29])
    for call in ("project", "project_full", "project_union"):
        want = getattr(tiny, call)(H, 4)
        got = getattr(tiny, call)(bad, 4)
        ids = got[0]
        assert ids.min() >= -1 and ids.max() < cfg.V, call
        if call != "project_union":      # the union's contents depend on every row's cluster
            assert np.array_equal(ids[good_rows], want[0][good_rows]), call
            assert np.array_equal(got[1][good_rows], want[1][good_rows]), call
        if call == "project":
            assert got[2].min() >= 0 and got[2].max() < cfg.K


def test_random_shapes(oracle):
    """Seeded random draws of (d, V, K, N, k) and ragged active sets, some of them empty, through every form
    of the projection against the oracle."""
    rs = np.random.default_rng(2208)
    for case in range(24):
        d = 8 * int(rs.integers(1, 257)) if case % 3 else int(rs.choice([8, 256, 512, 1024, 1536, 2048]))
        V = int(rs.integers(17, 5000))
        K = int(rs.integers(1, 300))
        N = int(rs.integers(1, 200))
        k = int(rs.choice([1, 2, 3, 4, 8, 13, 32]))
        sizes = rs.integers(0, min(V, 600) + 1, K)
        sizes[rs.random(K) < 0.1] = 0
        if sizes.sum() == 0:
            sizes[0] = 1
        print("random shapes: case %d  d %d V %d K %d N %d k %d" % (case, d, V, K, N, k), flush=True)
        r, W, b, C = _small_model(1000 + case, d, V, K)
        lists = [np.sort(r.choice(V, size=int(n), replace=False)) for n in sizes]
        off = np.zeros(K + 1, np.int64)
        np.cumsum(sizes, out=off[1:])
        ids = np.concatenate(lists).astype(np.int32)
        B = Built(W, b, C, off, ids, k_max=max(k, 1))
        H = _rows(r, C, N)
        ids_g, logp_g, g = B.project(H, k)
        g2, offs, z = B.debug(H)
        pu.check_projection(oracle, W, b, C, off, ids, H, k, ids_g, logp_g, g, logits_gpu=z, offs_gpu=offs)
        Hf = H[:64]
        f_ids, f_logp = B.project_full(Hf, k)
        pu.check_full(oracle, W, b, Hf, k, f_ids, f_logp)
        u_ids, u_logp, u_g, u_n = B.project_union(H, k)
        pu.check_union(oracle, W, b, C, off, ids, H, k, u_ids, u_logp, u_g, u_n)
        B.index.set_option("dispatch", 1)
        B.index.set_option("cost_bw_slab_gbs", 1)      # force the masked projection
        try:
            m_ids, m_logp, m_g = B.project(H, k)
            assert _planner_mode(B.index, N) == 1
        finally:
            B.index.set_option("cost_bw_slab_gbs", 6800)
            B.index.set_option("dispatch", 0)
        pu.check_projection(oracle, W, b, C, off, ids, H, k, m_ids, m_logp, m_g)
        del B


@pytest.mark.gpu
def test_small_batches_without_a_planning_kernel(oracle, tiny, mid):
    """Batches of at most 16 rows are planned by the projection workgroups themselves (no planning kernel,
    no item list): same plan as the planning kernel's, so the same bits, for every bucket structure, every
    number of loads in flight (which also sets how long the items are), and many calls in a row."""
    import torch
    r = np.random.default_rng(64)

    def run(B, H, k, small, dispatch, pf=0):
        B.index.set_option("small_path", small)
        B.index.set_option("small_pf", pf)
        B.index.set_option("dispatch", dispatch)
        try:
            out = B.project(H, k)
            return out, _planner_mode(B.index, H.shape[0]), _overflow(B.index, H.shape[0])
        finally:
            B.index.set_option("small_path", 1)
            B.index.set_option("small_pf", 0)
            B.index.set_option("dispatch", 0)

    for B in (tiny, mid):
        K = B.C.shape[0]
        for N, clusters in ((1, None), (2, [3, 3]), (3, [K - 1, 0, K - 1]), (5, None), (16, [1] * 16), (16, None),
                            (16, list(range(16))), (15, [7] * 8 + [2] * 7), (9, [4, 4, 4, 1, 1, 9, 9, 9, 9])):
            cl = None if clusters is None else [c % K for c in clusters]
            H = _rows(r, B.C, N, clusters=cl)
            for k in (1, 4, 8):
                print("small path:", B.cfg.name, "N", N, "k", k, flush=True)
                base, _, ovf0 = run(B, H, k, 0, 0)
                assert ovf0 == 0
                for pf in (0, 8, 16, 32):
                    got, _, ovf = run(B, H, k, 1, 0, pf)
                    assert ovf == 0
                    assert np.array_equal(got[2], base[2]) and np.array_equal(got[0], base[0])
                    if pf == 8:
                        assert np.array_equal(got[1], base[1]), "same item boundaries: same bits"
                    else:    # items sized for another number of resident workgroups: another order of the sums
                        assert np.allclose(got[1], base[1], rtol=0, atol=1e-5)
                pu.check_projection(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H, k, got[0], got[1], got[2])
                # with the planner free to choose the masked full projection
                d1, mode1, _ = run(B, H, k, 1, 1)
                d0, mode0, _ = run(B, H, k, 0, 1)
                assert np.array_equal(d1[0], d0[0]) and np.array_equal(d1[2], base[2])
                pu.check_projection(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H, k, d1[0], d1[1], d1[2])
    # several thousand calls in a row on one workspace
    H = _rows(r, tiny.C, 7)
    base = tiny.project(H, 2)
    Ht = tiny.rows(H)
    for i in range(2500):
        out = tiny.index.project(Ht, 2)
    torch.cuda.synchronize()
    assert np.array_equal(pu.to_np(out[0]), base[0]) and np.array_equal(pu.to_np(out[1]), base[1])
    # workspaces full of garbage: nothing in them is read before it is written
    need = (tiny.index.workspace_bytes(7) + 255) // 256 * 256
    big = torch.empty(40 * need, dtype=torch.uint8, device=tiny.dev)
    big.fill_(0x5A)
    outs = [tiny.index.project(Ht, 2, workspace=big[i * need:(i + 1) * need]) for i in range(40)]
    torch.cuda.synchronize()
    for i in (0, 1, 20, 39):
        assert np.array_equal(pu.to_np(outs[i][0]), base[0]) and np.array_equal(pu.to_np(outs[i][1]), base[1]), i
    del big, outs


@pytest.mark.gpu
def test_overlapping_calls_on_several_streams(tiny, mid):
    """Calls on different streams, each with a workspace and outputs of its own, may overlap on one index
    (nothing but the workspace and the outputs is written by a call): every result equals the one-stream result."""
    import torch
    for B, N, k in ((tiny, 3, 4), (mid, 2, 8), (mid, 40, 8)):
        dev = B.dev
        S, rounds = 4, 40
        Hs = [wl.make_rows(B.cfg, B.C, N=N, stream=500 + i)[0] for i in range(6)]
        want = [B.project(H, k) for H in Hs]
        hb = [B.rows(H) for H in Hs]
        streams = [torch.cuda.Stream(device=dev) for _ in range(S)]       # default priority
        wss = [torch.empty(B.index.workspace_bytes(N), dtype=torch.uint8, device=dev) for _ in range(S)]
        assert len({w.data_ptr() for w in wss}) == S
        outs = [[None] * rounds for _ in range(S)]
        torch.cuda.synchronize()
        for i in range(rounds):
            for si, st in enumerate(streams):
                with torch.cuda.stream(st):
                    outs[si][i] = B.index.project(hb[(i * S + si) % len(hb)], k, workspace=wss[si])
        torch.cuda.synchronize()
        for i in range(rounds):
            for si in range(S):
                w = want[(i * S + si) % len(hb)]
                got = outs[si][i]
                assert np.array_equal(pu.to_np(got[0]), w[0]) and np.array_equal(pu.to_np(got[1]), w[1]), (N, i, si)
                assert np.array_equal(pu.to_np(got[2]), w[2])


def _union_mode(index):
    """White-box: the planner's decision of the last vp_project_union call (header at the start of the workspace)."""
    import torch
    torch.cuda.synchronize()
    uws = index._uws[torch.cuda.current_stream().cuda_stream]
    return int(uws[:64].view(torch.int32)[7].item())


@pytest.mark.gpu
def test_union_form_either_way(oracle, tiny, mid):
    """The batch-union form gathers the columns of U, or, when U is large, runs the full projection with the
    boolean list as every row's mask: same results, both against the oracle's union mode."""
    r = np.random.default_rng(99)
    for B, N, k in ((tiny, 5, 4), (tiny, 16, 1), (tiny, 40, 4), (mid, 12, 8), (mid, 70, 8), (mid, 200, 2)):
        H, _q = wl.make_rows(B.cfg, B.C, N=N, stream=900 + N)
        print("union either way:", B.cfg.name, "N", N, "k", k, flush=True)
        B.index.set_option("union_dispatch", 0)
        try:
            gathered = B.project_union(H, k)
            assert _union_mode(B.index) == 0
        finally:
            B.index.set_option("union_dispatch", 1)
        B.index.set_option("cost_bw_gather_gbs", 1)          # make the gather look hopeless
        try:
            in_place = B.project_union(H, k)
            assert _union_mode(B.index) == 1
        finally:
            B.index.set_option("cost_bw_gather_gbs", 2400)
        for got in (gathered, in_place):
            pu.check_union(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H, k, got[0], got[1], got[2], got[3])
        assert np.array_equal(gathered[0], in_place[0]) and gathered[3] == in_place[3]
        assert np.allclose(gathered[1], in_place[1], rtol=0, atol=1e-4)
        default = B.project_union(H, k)
        assert np.array_equal(default[0], gathered[0])


@pytest.mark.gpu
@pytest.mark.parametrize("d, V", [(768, 20000), (1280, 12000)])
def test_union_form_where_the_columns_are_read_in_place(oracle, d, V):
    """The many-row kernel reads a small union's columns where they lie, in less time than one pass over a W of
    20,000 tokens: such a union is gathered, and one of most of the vocabulary is not."""
    r, W, b, C = _small_model(d, d, V, 8)
    for lo, hi, mode in ((40, 120, 0), (V // 3, V // 2, 1)):
        off, ids = _random_lists(r, 8, V, lo, hi)
        B = Built(W, b, C, off, ids, k_max=4)
        for N, k in ((17, 1), (65, 4)):
            H = _rows(r, C, N)
            print("union form: d", d, "V", V, "lists up to", hi, "N", N, "k", k, flush=True)
            got = B.project_union(H, k)
            assert _union_mode(B.index) == mode
            pu.check_union(oracle, W, b, C, off, ids, H, k, got[0], got[1], got[2], got[3])


@pytest.mark.gpu
def test_union_form_over_a_long_boolean_list(oracle):
    """More than 262,144 tokens: the boolean list spans many blocks of the three-step scan.  Gathered and
    in-place forms against the oracle."""
    r, W, b, C = _small_model(271, 16, 270000, 6)
    off, ids = _random_lists(r, 6, 270000, 300, 3000)
    B = Built(W, b, C, off, ids, k_max=4)
    for N, k in ((9, 2), (50, 4)):
        H = _rows(r, C, N)
        for dispatch, gbs in ((0, 2400), (1, 1)):
            print("large vocabulary union: N", N, "k", k, "in place" if dispatch else "gathered", flush=True)
            B.index.set_option("union_dispatch", dispatch)
            B.index.set_option("cost_bw_gather_gbs", gbs)
            try:
                got = B.project_union(H, k)
                assert _union_mode(B.index) == dispatch
            finally:
                B.index.set_option("union_dispatch", 1)
                B.index.set_option("cost_bw_gather_gbs", 2400)
            pu.check_union(oracle, W, b, C, off, ids, H, k, got[0], got[1], got[2], got[3])


@pytest.mark.gpu
def test_item_order_of_plans_with_heavy_buckets(oracle, tiny, mid):
    """A bucket of more than four row groups switches the workgroup -> item map to blocks of consecutive items
    per XCD with different starting points; every item must still be done exactly once."""
    import torch
    r = np.random.default_rng(7)
    for B, N, heavy in ((tiny, 200, 120), (tiny, 1000, 1000), (mid, 300, 90), (mid, 81, 81)):
        K = B.C.shape[0]
        clusters = np.concatenate([np.full(heavy, 3 % K), r.integers(0, K, N - heavy)]).astype(np.int64)
        r.shuffle(clusters)
        H = _rows(r, B.C, N, clusters=clusters)
        for k in (1, 4):
            print("heavy bucket:", B.cfg.name, "N", N, "rows in one cluster", heavy, "k", k, flush=True)
            ids, logp, g = B.project(H, k)
            ws = B.index.workspace(N)
            torch.cuda.synchronize()
            hdr = ws[:64].view(torch.int32)[:8].tolist()
            assert hdr[4] == -32 and hdr[7] == 0, hdr          # the swizzle of clustered plans is on
            pu.check_projection(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H, k, ids, logp, g)


# ------------------------------------------------- the largest shapes, every form, and repeatability
def _points_check(oracle, B, H, k, ids, logp):
    """Every returned (row, token) against the oracle's own logit of that pair (Eq. 1): each row's logits
    descend, equal logits keep ascending token ids, and log-prob differences within a row equal logit
    differences (the log-sum-exp cancels).  Works at any size: one inner product per returned entry."""
    N = H.shape[0]
    rows = np.repeat(np.arange(N, dtype=np.int32), k)
    toks = ids.reshape(-1).astype(np.int32)
    assert np.all((toks >= 0) & (toks < B.W.shape[1]))
    z = oracle.logit_points(B.W, B.b, H, rows, toks).reshape(N, k)
    assert np.all(z[:, :-1] >= z[:, 1:] - pu.TAU), "logits of a row's entries do not descend"
    tie = z[:, :-1] == z[:, 1:]
    assert np.all(ids[:, :-1][tie] < ids[:, 1:][tie])
    for r in range(N):
        assert len(set(ids[r].tolist())) == k
    d_logp = logp[:, :1].astype(np.float64) - logp.astype(np.float64)
    d_z = z[:, :1] - z
    err = np.abs(d_logp - d_z).max()
    assert err <= pu.SANITY, "log-prob differences off by %g" % err
    return float(err)


def test_full_projection_at_the_largest_shapes(oracle, large, skewed):
    """vp_project_full at the sweep's 1,024 rows and at the skewed workload's 4,096 rows of d = 1,536: every
    returned entry against the oracle's logit of that (row, token), and whole rows (log-softmax over V, top-k)
    for a sample the oracle can afford."""
    cases = ((large, wl.CONFIGS["sweep"], 1024, 1), (large, wl.CONFIGS["sweep"], 1024, 8),
             (skewed, skewed.cfg, skewed.cfg.N, skewed.cfg.k))
    for B, cfg, N, k in cases:
        H, q = wl.make_rows(cfg, B.C, N=N, stream=33)
        ids, logp = B.project_full(H, k)
        assert _overflow(B.index, N) == 0
        err = _points_check(oracle, B, H, k, ids, logp)
        sample = np.array([0, 1, N // 3, N // 2, N - 65, N - 64, N - 2, N - 1])
        st = pu.check_full(oracle, B.W, B.b, H[sample], k, ids[sample], logp[sample])
        print("full projection", cfg.name, N, k, "points err", err, st, flush=True)
        ids2, logp2 = B.project_full(H, k)
        assert np.array_equal(ids, ids2) and np.array_equal(logp, logp2), "two runs differ"


def _masked(B, H, k, force=True):
    """vp_project with the planner switched on; force: the slabs made to look hopeless, so that the masked
    full projection is taken whatever the batch."""
    B.index.set_option("dispatch", 1)
    if force:
        B.index.set_option("cost_bw_slab_gbs", 1)
    try:
        out = B.project(H, k)
        return out, _planner_mode(B.index, H.shape[0]), _overflow(B.index, H.shape[0])
    finally:
        B.index.set_option("cost_bw_slab_gbs", 6800)
        B.index.set_option("dispatch", 0)


def test_every_form_on_the_large_and_skewed_indexes(oracle, large, skewed):
    """The masked full projection and the batch-union form at the sizes the benchmark runs them: N = 256 on the
    large index (items of 64 rows, rows in LDS) and N = 4,096 at d = 1,536 (items of 48 rows).  Same token ids
    as the per-cluster slabs, log-probs within 1e-4 of them, sampled rows against the oracle; the union of 226
    active sets with random top-up ids is the whole vocabulary, so that form must equal the full projection."""
    for B, cfg in ((large, large.cfg), (skewed, skewed.cfg)):
        N, k = cfg.N, cfg.k
        H, q = wl.make_rows(cfg, B.C, N=N, stream=44)
        base = B.project(H, k)
        assert _overflow(B.index, N) == 0
        (m_ids, m_logp, m_g), mode, ovf = _masked(B, H, k)
        assert mode == 1 and ovf == 0
        assert np.array_equal(m_g, base[2]) and np.array_equal(m_ids, base[0])
        assert np.allclose(m_logp, base[1], rtol=0, atol=1e-4)
        sample = np.array([0, 5, N // 2, N - 1, int(np.argmax(np.bincount(q)[q]))])   # incl. a row of the fullest bucket
        st = pu.check_projection(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H[sample], k, m_ids[sample],
                                 m_logp[sample], m_g[sample])
        print("masked", cfg.name, st, flush=True)
        # the planner left to itself: whichever form it takes, the same results
        (d_ids, d_logp, d_g), mode, ovf = _masked(B, H, k, force=False)
        assert ovf == 0 and np.array_equal(d_ids, base[0]) and np.allclose(d_logp, base[1], rtol=0, atol=1e-4)
        print("planner chose", cfg.name, mode, flush=True)
        # twice the same call: the same bits, in every form
        for fn in (lambda: B.project(H, k), lambda: _masked(B, H, k)[0], lambda: B.project_union(H, k)[:2]):
            a, b2 = fn(), fn()
            assert np.array_equal(a[0], b2[0]) and np.array_equal(a[1], b2[1]), "two runs differ"
        u_ids, u_logp, u_g, nu = B.project_union(H, k)
        lists = [B.cand_ids[B.cand_off[j]:B.cand_off[j + 1]] for j in np.unique(u_g)]
        U = np.unique(np.concatenate(lists))
        assert nu == U.size and np.array_equal(u_g, base[2])
        if U.size == B.W.shape[1]:
            f_ids, f_logp = B.project_full(H, k)
            assert np.array_equal(u_ids, f_ids) and np.allclose(u_logp, f_logp, rtol=0, atol=1e-4)
        else:
            _points_check(oracle, B, H, k, u_ids, u_logp)
            assert np.all(np.isin(u_ids, U))


def test_debug_logits_on_skewed_rows(oracle, skewed):
    """Candidate logits at d = 1,536, element by element, for rows of the fullest and of ordinary buckets."""
    cfg = skewed.cfg
    H, q = wl.make_rows(cfg, skewed.C)
    heavy = int(np.argmax(np.bincount(q, minlength=cfg.K)))
    pick = np.concatenate([np.nonzero(q == heavy)[0][:20], np.nonzero(q != heavy)[0][:12]])
    print("skewed logits", _full_check(oracle, skewed, H[pick], cfg.k, with_logits=True))


def test_library_defaults_on_all_five_workloads(oracle, tiny, mid, large, skewed):
    """The call as shipped (the planner free to choose the form) on every configured workload: all rows against
    the oracle where it can afford them, a sample elsewhere, plus the returned entries' own logits for all rows."""
    sweep = wl.CONFIGS["sweep"]
    for B, cfg, N, k in ((tiny, tiny.cfg, None, None), (mid, mid.cfg, None, None), (large, large.cfg, None, None),
                         (large, sweep, 64, 1), (large, sweep, 1024, 1), (skewed, skewed.cfg, None, None)):
        N, k = N or cfg.N, k or cfg.k
        H, q = wl.make_rows(cfg, B.C, N=N, stream=55)
        (ids, logp, g), mode, ovf = _masked(B, H, k, force=False)
        assert ovf == 0
        sample = np.arange(N) if N <= 64 else np.unique(np.linspace(0, N - 1, 12).astype(int))
        st = pu.check_projection(oracle, B.W, B.b, B.C, B.cand_off, B.cand_ids, H[sample], k, ids[sample],
                                 logp[sample], g[sample])
        g_or, excused = pu.check_clusters(oracle, H, B.C, g)
        err = _points_check(oracle, B, H, k, ids, logp) if min(B.cand_off[1:] - B.cand_off[:-1]) >= k else None
        print("defaults", cfg.name, N, k, "mode", mode, st, "excused clusters", excused, "points", err, flush=True)


def _time_calls(B, Ht, k, steps=20):
    import time
    import torch
    ws = B.index.workspace(Ht.shape[0])
    # ten milliseconds of the same calls first: after a pause on the host the first calls run up to 10 % slower
    # than the steady state, which would be charged to whichever form is timed first
    t_w = time.perf_counter()
    while time.perf_counter() - t_w < 0.010:
        for i in range(8):
            B.index.project(Ht, k, workspace=ws)
        torch.cuda.synchronize()
    best = float("inf")
    for rep in range(3):
        for i in range(3):
            B.index.project(Ht, k, workspace=ws)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(steps):
            B.index.project(Ht, k, workspace=ws)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / steps)
    return best


def test_planner_picks_the_faster_form(tiny, mid, large, skewed):
    """The cost model against the clock, over k-extents 512 / 1,024 / 1,536, batch sizes and occupancies (rows
    spread over the clusters, or crowded into a few): the planner's own choice must run within 10 % (plus a few
    microseconds of timer noise) of the faster of the two forms, each forced through the same planner."""
    r = np.random.default_rng(91)
    report = []
    for B, sizes in ((tiny, (16, 64, 512)), (mid, (24, 64, 200)), (large, (20, 32, 256)), (skewed, (64, 1024, 4096))):
        K = B.C.shape[0]
        for N in sizes:
            for spread in ("all clusters", "four clusters"):
                clusters = None if spread == "all clusters" else r.integers(0, K, 4)[r.integers(0, 4, N)]
                Ht = B.rows(_rows(r, B.C, N, clusters=clusters))
                k = B.cfg.k
                t = {}
                B.index.set_option("dispatch", 1)
                try:
                    t["planner"] = _time_calls(B, Ht, k)
                    mode = _planner_mode(B.index, N)
                    B.index.set_option("cost_bw_slab_gbs", 1)          # slabs look hopeless: masked full projection
                    t["masked"] = _time_calls(B, Ht, k)
                    assert _planner_mode(B.index, N) == 1 or N <= 16
                    B.index.set_option("cost_bw_slab_gbs", 6800)
                    full = (5100, 17000, 14000, 8000)
                    for name in ("cost_bw_full_gbs", "cost_bw_l2_gbs", "cost_bw_gemm_gbs", "cost_bw_gemm_split_gbs"):
                        B.index.set_option(name, 1)                    # the full projection looks hopeless: slabs
                    t["slabs"] = _time_calls(B, Ht, k)
                    assert _planner_mode(B.index, N) == 0
                finally:
                    for name, v in zip(("cost_bw_full_gbs", "cost_bw_l2_gbs", "cost_bw_gemm_gbs", "cost_bw_gemm_split_gbs"),
                                       (5100, 17000, 14000, 8000)):
                        B.index.set_option(name, v)
                    B.index.set_option("cost_bw_slab_gbs", 6800)
                    B.index.set_option("dispatch", 0)
                best = min(t["masked"], t["slabs"])
                report.append((B.cfg.name, N, spread, mode, t))
                print("planner", B.cfg.name, N, spread, "chose", mode, {n: round(v * 1e6, 1) for n, v in t.items()}, flush=True)
                assert t["planner"] <= 1.10 * best + 6e-6, (B.cfg.name, N, spread, mode, t)


def test_index_without_the_token_major_copy(oracle):
    """VP_BUILD_NO_UNION: a smaller arena, vp_project and vp_project_full as ever, vp_project_union refused."""
    torch = _torch()
    from paper_2208_06874_amd import vp
    r, W, b, C = _small_model(21, 256, 4000, 6)
    off, ids = _random_lists(r, 6, 4000, 100, 600)
    dev = torch.device("cuda:0")
    Wt, bt, Ct = (torch.from_numpy(a).to(dev) for a in (W, b, C))
    full = vp.vp_build(Wt, bt, Ct, off, ids, k_max=4)
    lean = vp.vp_build(Wt, bt, Ct, off, ids, k_max=4, flags=vp.BUILD_NO_UNION)
    assert full.info()["arena_bytes_used"] - lean.info()["arena_bytes_used"] >= 4000 * 256 * 2
    H = _rows(r, C, 40)
    Ht = torch.from_numpy(H).to(dev)
    a_ids, a_logp, a_g = full.project(Ht, 4)
    b_ids, b_logp, b_g = lean.project(Ht, 4)
    torch.cuda.synchronize()
    assert torch.equal(a_ids, b_ids) and torch.equal(a_logp, b_logp) and torch.equal(a_g, b_g)
    pu.check_projection(oracle, W, b, C, off, ids, H, 4, pu.to_np(b_ids), pu.to_np(b_logp), pu.to_np(b_g))
    f_ids, f_logp = lean.project_full(Ht, 4)
    torch.cuda.synchronize()
    pu.check_full(oracle, W, b, H, 4, pu.to_np(f_ids), pu.to_np(f_logp))
    with pytest.raises(vp.VpError) as e:
        lean.project_union(Ht, 4)
    assert e.value.status == vp.VP_ERR_UNSUPPORTED and "NO_UNION" in str(e.value)


VP_FLOOR_NONE = 0x007fffff


def _rows_that_traded(index, N, K):
    """(rows whose items traded the bests of sets in the last many-row call, the plan's records by position) from the workspace: the
    planner sets a row's eight bounds to the key of -infinity, a trade raises those of the sets that have a candidate."""
    ws = index.workspace(N)
    up = lambda x: (x + 255) // 256 * 256
    at = 128 + (128 + up(36 * N) - 32 * N) // 128 * 128
    bounds = pu.to_np(ws[at:at + 32 * N]).view(np.uint32).reshape(N, 8)
    at = 256 + up(36 * N) + up(N * ((K + 15) // 16) * 8) + 2 * up(4 * N)
    plan = pu.to_np(ws[at:at + 32 * N]).view(np.int32).reshape(N, 8)
    return (bounds != VP_FLOOR_NONE).any(1), plan


def _tied_ids_in_order(ids, tied):
    """Of the tokens with one and the same logit a row lists the smallest ones, ascending."""
    for row in ids:
        mine = row[np.isin(row, tied)]
        assert np.array_equal(mine, tied[:len(mine)]), (row, tied[:8])


ALL = (4, 6, 8)


@pytest.mark.parametrize("d,N,groups,items,trades", [
    (256, 64, 36, 26, (8,)), (256, 64, 32, 25, ALL), (256, 64, 48, 24, ()), (256, 127, 144, 25, (6, 8)), (512, 64, 36, 25, (8,)), (512, 64, 56, 25, ALL), (512, 52, 56, 22, ()),
    (768, 64, 36, 25, ()), (768, 192, 16, 25, ALL), (1024, 47, 36, 26, ()), (1024, 60, 28, 25, ()), (1024, 60, 32, 25, ALL),
    (1024, 64, 68, 25, (8,)), (1024, 130, 36, 25, ALL), (1280, 48, 20, 25, (8,)), (1280, 96, 36, 25, ()), (1280, 100, 36, 25, (8,)), (1536, 36, 24, 25, ()),
    (1536, 37, 28, 25, ALL), (1536, 48, 52, 25, ALL)])
def test_bests_of_sets_traded_between_many_items(oracle, d, N, groups, items, trades):
    """Rows whose candidates are spread over many items trade the bests of eight sets of candidates before the first list entry: by
    width, list length, row groups and steps (vp_trades_sets), from 24 full items on, with three quarters of the row slots
    in use, and in no item of a call that does not (trades: the list lengths among 4, 6 and 8 that do).  A third of the
    vocabulary ties, in every set and item; a row with a few candidates only; a last item in which wavefronts have no step;
    steps of two groups and of four, one row group and several; plain and masked, twice to the bit."""
    V = 16 * groups * items - 16 * min(groups - 13, 60) - 5   # (the last item: 12 groups and a piece, or some more)
    r, W, b, C = _small_model(70 + d + N, d, V, 3)
    W[:, ::3] = W[:, :1]                     # the same logit, whatever the row, somewhere among or near the best ones
    b[::3] = np.float16(3.5)
    off, ids = _random_lists(r, 3, V, 2, 9)
    full = np.sort(r.choice(V, size=V // 2, replace=False)).astype(np.int32)
    ids = np.concatenate([full, ids[off[1]:]]).astype(np.int32)
    off = np.concatenate([[0], off[1:] - off[1] + len(full)]).astype(np.int64)
    B = Built(W, b, C, off, ids, k_max=9)
    per = 64 if d <= 1024 else 48
    rgs = (N + per - 1) // per
    H = _rows(r, C, N)
    # (a last row group of a few rows does not trade)
    full_groups = np.arange(N) // per < rgs - (rgs > 1 and 0 < 4 * (N % per) < 3 * per)
    B.index.set_option("gemm_lds_items", items * rgs)
    for k in (3, 4, 6, 8, 9):
        got = B.project_full(H, k)
        ws = B.index.workspace(N)[:64].view(_torch().int32)
        assert ws[0].item() == items * rgs and ws[1].item() * 4 == groups, (ws[0].item(), ws[1].item())
        traded, _ = _rows_that_traded(B.index, N, 3)
        assert np.array_equal(traded, full_groups if k in trades else np.full(N, False)), (k, traded)
        again = B.project_full(H, k)
        for x, y in zip(got, again):
            assert np.array_equal(x, y)
        pu.check_full(oracle, W, b, H, k, *got)
        _tied_ids_in_order(got[0], np.arange(0, V, 3))
        if k in (3, 9):
            continue
        got, mode, ovf = _masked(B, H, k)
        assert mode == 1 and ovf == 0
        traded, _ = _rows_that_traded(B.index, N, 3)
        big = got[2] == 0                    # (rows of the long list: the others' few candidates may all be seen later than the first step)
        assert np.array_equal(traded[big], full_groups[big] & (k in trades)), (k, traded)
        pu.check_projection(oracle, W, b, C, off, ids, H, k, *got)
        _tied_ids_in_order(got[0][big], full[full % 3 == 0])


def test_bests_of_sets_traded_in_a_plan_of_several_forms(oracle):
    """Masked rows among rows on slabs: a masked row's sets are found by its number, not by its place in the plan, and begin anew
    in every call (the call before it had larger logits in the same workspace)."""
    d, V, K, N, k = 512, 40000, 40, 400, 8
    r, W, b, C = _small_model(77, d, V, K)
    off, ids = _random_lists(r, K, V, 200, 1500)
    B = Built(W, b, C, off, ids)
    p = np.arange(1, K + 1) ** -1.3
    q = r.choice(r.permutation(K), size=N, p=p / p.sum())
    q[:K] = np.arange(K)
    H = _rows(r, C, N, clusters=q)
    base = B.project(H, k)
    B.index.set_option("dispatch", 1)
    rates = {"cost_row_slab_ns": 0, "cost_bw_l2_gbs": 1000000, "cost_bw_full_gbs": 1000000, "cost_bw_slab_gbs": 2, "cost_bw_gemm_gbs": 14}
    for name, v in rates.items():
        B.index.set_option(name, v)
    larger = B.project((H.astype(np.float32) * 4).astype(np.float16), k)
    assert (larger[2] == base[2]).mean() > 0.9
    got = B.project(H, k)
    assert _planner_mode(B.index, N) == 2 and _overflow(B.index, N) == 0
    traded, plan = _rows_that_traded(B.index, N, K)
    masked = plan[plan[:, 5] == -1, 0]
    assert len(masked) > 64 and len(masked) < N and traded[masked].sum() >= 64, (len(masked), traded[masked].sum())
    assert not np.array_equal(masked, np.sort(masked))           # (the plan's order is not the rows')
    again = B.project(H, k)
    for x, y in zip(got, again):
        assert np.array_equal(x, y)
    assert np.array_equal(got[0], base[0]) and np.array_equal(got[2], base[2])
    assert np.allclose(got[1], base[1], rtol=0, atol=1e-4)
    pu.check_projection(oracle, W, b, C, off, ids, H, k, *got)


def test_crowded_clusters_do_not_trade(oracle):
    """Crowded clusters' items run beside masked rows' in kernels that trade, without the code that does, however long their lists:
    three clusters of 13,000 tokens with sixty rows each, a fourth of two rows."""
    d, V, K, k = 512, 60000, 4, 8
    r, W, b, C = _small_model(78, d, V, K)
    lists = [np.sort(r.choice(V, size=n, replace=False)) for n in (13000, 13000, 13000, 400)]
    off = np.cumsum([0] + [len(x) for x in lists]).astype(np.int64)
    ids = np.concatenate(lists).astype(np.int32)
    B = Built(W, b, C, off, ids)
    q = r.permutation(np.r_[np.repeat([0, 1, 2], 60), 3, 3])
    N = len(q)
    H = _rows(r, C, N, clusters=q)
    base = B.project(H, k)
    B.index.set_option("dispatch", 1)
    for name, v in {"cost_row_slab_ns": 0, "cost_bw_slab_gbs": 7, "cost_bw_l2_gbs": 17, "cost_bw_full_gbs": 5, "cost_bw_gemm_gbs": 14}.items():
        B.index.set_option(name, v)
    got = B.project(H, k)
    assert _planner_mode(B.index, N) == 2 and _overflow(B.index, N) == 0
    assert int(B.index.workspace(N)[:64].view(_torch().int32)[12].item()) >= 3 * 24     # (their items)
    traded, plan = _rows_that_traded(B.index, N, K)
    crowded = plan[np.isin(plan[:, 1], (0, 1, 2)), 0]
    assert len(crowded) == 180 and not traded[crowded].any()
    assert np.array_equal(got[0], base[0]) and np.array_equal(got[2], base[2])
    assert np.allclose(got[1], base[1], rtol=0, atol=1e-4)
    pu.check_projection(oracle, W, b, C, off, ids, H, k, *got)


@pytest.mark.parametrize("N,K", [(65, 40), (256, 1300), (333, 1990), (769, 1990), (2047, 2000)])
def test_every_form_of_the_many_row_eq2_kernel_in_decoding(oracle, N, K):
    """One or two row tiles x one to eight centroid tiles per wavefront, by how many workgroups each leaves (the sixth form, one
    row tile x eight, serves the training alone): a last row tile and a last centroid tile that are not full, duplicate
    centroids (ties to the lowest), a width that ends inside a k-tile."""
    d, V = 264, 300
    r, W, b, C = _small_model(90 + N, d, V, K)
    C[K // 2:K // 2 + 9] = C[3]
    off, ids = _random_lists(r, K, V, 4, 12)
    B = Built(W, b, C, off, ids)
    H = _rows(r, C, N, clusters=np.concatenate([np.full(20, 3), r.integers(0, K, N - 20)]))
    got = B.project(H, 2)
    assert (got[2][:20] == 3).all()
    pu.check_projection(oracle, W, b, C, off, ids, H, 2, *got)


@pytest.mark.parametrize("k", [1, 2, 4, 5, 8, 9])
def test_merge_of_equal_logits_over_many_parts(oracle, k):
    """Rows of more parts than a workgroup of the merge has threads, of a few hundred and of at most a wavefront's lanes: forty
    tokens, spread over the parts, share a row's largest logit, and the k smallest of them win, in order."""
    d, V = 64, 40000
    r, W, b, C = _small_model(5 + k, d, V, 1)
    W[:] = W[:, :1]
    b[:] = b[0]
    best = np.sort(r.choice(V, 40, replace=False))
    b[best] += np.float16(2.0)
    B = Built(W, b, C, np.array([0, V], np.int64), np.arange(V, dtype=np.int32), k_max=16)
    H = _rows(r, C, 2)
    for wanted, least, most in ((2048, 257, 2048), (200, 65, 256), (16, 9, 64)):
        B.index.set_option("full_target_items", wanted)
        got = B.project_full(H, k)
        parts = B.index.workspace(2)[:64].view(_torch().int32)[0].item()
        assert least <= parts <= most, parts
        assert np.array_equal(got[0], np.tile(best[:k], (2, 1))), (wanted, got[0], best[:k])
        assert (got[1] == got[1][:, :1]).all()
        pu.check_full(oracle, W, b, H, k, *got)


@pytest.mark.parametrize("d,groups", [(256, 16), (256, 20), (512, 12), (512, 32), (768, 32), (1024, 64), (1024, 68), (1280, 20), (1280, 24),
                                      (1536, 32), (1536, 36)])
def test_steps_of_one_two_and_four_groups(oracle, d, groups):
    """Single row groups at both sides of the lines between steps of one, two and four candidate groups, plain and masked: a last
    item of another length, rows and candidates that fill no tile, d inside a k-tile."""
    items, N = 5, 33
    V = 16 * groups * items - 16 * 6 - 3
    r, W, b, C = _small_model(500 + d + groups, d - 8, V, 3)
    off, ids = _random_lists(r, 3, V, V // 3, V // 2)
    B = Built(W, b, C, off, ids, k_max=9)
    B.index.set_option("gemm_lds_items", items)
    H = _rows(r, C, N)
    for k in (1, 2, 5, 9):
        got = B.project_full(H, k)
        ws = B.index.workspace(N)[:64].view(_torch().int32)
        assert ws[0].item() == items and ws[1].item() * 4 == groups
        pu.check_full(oracle, W, b, H, k, *got)
        got, mode, ovf = _masked(B, H, k)
        assert mode == 1 and ovf == 0
        pu.check_projection(oracle, W, b, C, off, ids, H, k, *got)


@pytest.mark.parametrize("d,N,groups,items", [(256, 64, 36, 26), (1024, 64, 36, 25), (256, 128, 144, 24), (256, 20, 36, 10)])
def test_nan_candidate_costs_no_other_candidate_its_place(oracle, d, N, groups, items):
    """One token's bias is NaN (its logit is, and so is the row's log-sum-exp); eight others are far ahead of all the rest, one
    of them among the sixteen candidates that the same lane of the many-row kernel folds.  The eight are the top-8 all the
    same: NaN is never listed and costs no other candidate its place, whether or not items trade the bests of sets of candidates (which know the
    eight from the first step on)."""
    V = 16 * groups * items
    r, W, b, C = _small_model(300 + d + N, d, V, 2)
    nan_at = 16 * groups * 3                                 # the first candidate of the fourth item
    # (one in each of the eight sets: lane quarter s % 4, of the first wavefront or the second)
    top = np.array([nan_at + 1] + [16 * groups * ((s + 3) % items) + 4 * (s % 4) + 64 * (s // 4) + 2 for s in range(1, 8)])
    b[top] = np.float16(60.0) + np.arange(8).astype(np.float16)
    b[nan_at] = np.nan
    B = Built(W, b, C, np.array([0, V, V + 9], np.int64), np.concatenate([np.arange(V), np.arange(9)]).astype(np.int32), k_max=9)
    per = 64
    B.index.set_option("gemm_lds_items", items * ((N + per - 1) // per))
    H = _rows(r, C, N, clusters=np.zeros(N, int))
    for form in ("full", "masked"):
        for k in (8, 9, 4):
            if form == "full":
                ids, logp = B.project_full(H, k)
            else:
                (ids, logp, g), mode, ovf = _masked(B, H, k)
                assert mode == 1 and ovf == 0 and (g == 0).all()
            assert np.isnan(logp).all(), (form, k)
            if k >= 8:
                assert np.array_equal(np.sort(ids[:, :8], axis=1), np.tile(np.sort(top), (N, 1))), (form, k, ids[0], top)
            assert (ids >= 0).all() and not (ids == nan_at).any() and (np.isin(ids[:, :4], top)).all()
