"""GPU parity of the k-nearest-neighbour graph construction (Section III-A) against the oracle, through the C ABI:
the exact search, the list of undirected edges, and the chain points -> neighbours -> edges -> CSR."""
import numpy as np
import pytest

from oracle import knn as oknn
from paper_1802_04450_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1802_04450_amd import binding
    binding.lib()
    return binding


def _dev(a, dtype):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda:0")


def _check_search(B, x, k):
    ref_i, ref_d = oknn.knn_bruteforce(x, k)
    idx, dist = B.sc_knn_search(_dev(x, torch.float64), k)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    # the neighbour sets are integers decided by fp64 distances on both sides: equal unless two candidates of one
    # query are closer than the rounding of the sum, which the distances themselves then show
    same = idx == ref_i
    if not same.all():
        bad = np.argwhere(~same)
        for i, a in bad:
            assert abs(dist[i, a] - ref_d[i, a]) <= 4e-15 * max(ref_d[i, a], 1e-300), (i, a)
        assert len(bad) <= 2 * max(1, x.shape[0] // 1000)
    np.testing.assert_allclose(dist, ref_d, rtol=1e-13, atol=0)
    return idx, dist


# several workgroups of 128 queries and a ragged last one; candidate counts not a multiple of 4; padded and unpadded
# dimensions; k from 1 to all the other points
@pytest.mark.parametrize("n,d,k", [(1500, 5, 7), (1003, 3, 1), (130, 33, 20), (641, 16, 10), (20, 2, 19), (2, 1, 1),
                                   (515, 128, 10), (300, 8, 32), (300, 130, 5), (700, 64, 12), (333, 100, 3),
                                   # many workgroups, many candidate tiles
                                   (8300, 8, 5), (8450, 32, 12), (9001, 13, 10)])
def test_search_matches_oracle(B, n, d, k):
    rng = np.random.default_rng(100 * n + d)
    x = rng.standard_normal((n, d)) * rng.uniform(0.5, 2.0, size=(1, d))
    idx, dist = _check_search(B, x, k)
    assert np.all(idx != np.arange(n)[:, None]) and np.all(np.diff(dist, axis=1) >= 0)


# the bf16 screen: its smallest sizes, ragged tiles of 32 points and of 512 queries, every padded dimension, k up to the
# most that fits; neighbours that follow one another in memory; a common offset; points that the screen cannot tell apart
@pytest.mark.parametrize("n,d,k,kind", [(512, 3, 31, "random"), (513, 70, 7, "random"), (2048, 16, 10, "random"), (2049, 1, 1, "random"), (2111, 128, 20, "random"),
                                        (4097, 17, 32, "random"), (3600, 64, 200, "random"), (6000, 33, 20, "sorted"),
                                        (5003, 32, 15, "offset"), (2500, 12, 8, "copies"), (4000, 3, 10, "far"),
                                        (2600, 8, 5, "equal"), (2300, 10, 6, "tiny")])
def test_screened_search_matches_oracle(B, n, d, k, kind):
    rng = np.random.default_rng(7 * n + d)
    x = rng.standard_normal((n, d))
    if kind == "sorted":          # clusters, each contiguous
        x += 30.0 * rng.standard_normal((12, d))[np.arange(n) * 12 // n]
    elif kind == "offset":
        x += 1e6
    elif kind == "copies":        # more equal points than a list holds, beside ordinary ones
        x[::3] = x[0]
    elif kind == "far":           # spread 1e6, distances 1e-3: below the resolution of the screen
        x = 1e6 * rng.standard_normal((40, d))[rng.integers(0, 40, n)] + 1e-3 * x
    elif kind == "equal":
        x[:] = x[0]
    elif kind == "tiny":
        x *= 1e-150
    ref_i, ref_d = oknn.knn_bruteforce(x, k)
    idx, dist = B.sc_knn_search(_dev(x, torch.float64), k)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    # candidates are ranked by the fp64 sum of squared differences on both sides, in coordinate order here and in the
    # oracle's own order there: two whose sums agree to the rounding of d + 2 additions may change places
    bad = idx != ref_i
    assert np.all(np.abs(dist - ref_d)[bad] <= (d + 2) * 2.3e-16 * ref_d[bad])
    np.testing.assert_allclose(dist, ref_d, rtol=1e-13, atol=0)
    assert np.all(idx != np.arange(n)[:, None])


# whole coordinates: distances are exact and many are equal, in their upper words or altogether.  Lists of one and of several waves'
# lengths, on both sides of where a workgroup has one wave (170 neighbours); coordinates that fill no piece of 8, 16 or 32
@pytest.mark.parametrize("n,d,k,most", [(4000, 2, 10, 60), (4000, 2, 64, 60), (4003, 5, 33, 12), (4000, 18, 170, 9), (4000, 18, 171, 9),
                                        (4100, 36, 20, 400), (4001, 128, 40, 3), (6000, 3, 200, 25), (3000, 40, 1, 100_000)])
def test_screened_search_ranks_equal_distances_by_index(B, n, d, k, most):
    rng = np.random.default_rng(n + d + k)
    x = rng.integers(0, most, size=(n, d)).astype(np.float64)
    sq = (x * x).sum(axis=1)
    d2 = sq[:, None] + sq[None, :] - 2.0 * (x @ x.T)    # whole numbers below 2^53: exact
    np.fill_diagonal(d2, np.inf)
    near = np.argsort(d2, axis=1, kind="stable")[:, :k]
    idx, dist = B.sc_knn_search(_dev(x, torch.float64), k)
    np.testing.assert_array_equal(idx.cpu().numpy(), near)
    np.testing.assert_array_equal(dist.cpu().numpy(), np.sqrt(np.take_along_axis(d2, near, axis=1)))


def test_search_orders_equal_distances_by_index(B):
    # integer points on a line and on a small grid: many exactly equal distances, all sums exact in fp64
    x = np.arange(37, dtype=np.float64)[:, None]
    ref_i, ref_d = oknn.knn_bruteforce(x, 6)
    idx, dist = B.sc_knn_search(_dev(x, torch.float64), 6)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref_i)
    np.testing.assert_array_equal(dist.cpu().numpy(), ref_d)
    g = np.stack(np.meshgrid(np.arange(13.0), np.arange(11.0), indexing="ij"), axis=-1).reshape(-1, 2)
    ref_i, ref_d = oknn.knn_bruteforce(g, 8)
    idx, dist = B.sc_knn_search(_dev(g, torch.float64), 8)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref_i)
    np.testing.assert_array_equal(dist.cpu().numpy(), ref_d)


def test_search_strided_rows_and_errors(B):
    rng = np.random.default_rng(2)
    n, d, k = 700, 6, 5
    big = torch.as_tensor(rng.standard_normal((n, 9)), device="cuda:0")
    x = big[:, :d]                                   # leading dimension 9: through the C ABI directly
    lib = B.lib()
    st = torch.cuda.current_stream().cuda_stream
    io = torch.empty((n, k), dtype=torch.int32, device="cuda:0")
    do = torch.empty((n, k), dtype=torch.float64, device="cuda:0")
    assert lib.sc_knn_search(x.data_ptr(), 9, n, d, k, io.data_ptr(), do.data_ptr(), st) == 0
    ref_i, ref_d = oknn.knn_bruteforce(big.cpu().numpy()[:, :d], k)
    np.testing.assert_array_equal(io.cpu().numpy(), ref_i)
    np.testing.assert_allclose(do.cpu().numpy(), ref_d, rtol=1e-13)
    assert lib.sc_knn_search(x.data_ptr(), 9, n, d, n, io.data_ptr(), do.data_ptr(), st) == -2      # k_nn > n - 1
    assert lib.sc_knn_search(x.data_ptr(), 5, n, d, k, io.data_ptr(), do.data_ptr(), st) == -2      # ldx < d
    assert lib.sc_knn_search(x.data_ptr(), 9, 1, d, 1, io.data_ptr(), do.data_ptr(), st) == -2      # one point
    assert lib.sc_knn_search(0, 9, n, d, k, io.data_ptr(), do.data_ptr(), st) == -1                 # null pointer
    assert lib.sc_knn_search(x.data_ptr(), 9, n, 6, 250, io.data_ptr(), do.data_ptr(), st) == -2    # LDS: k_nn too large


@pytest.mark.parametrize("n,d,k,sigma", [(1200, 4, 6, 0.0), (777, 10, 15, 1.3), (50, 2, 49, 0.5)])
def test_union_pairs_match_oracle(B, n, d, k, sigma):
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, d))
    ref_i, ref_d = oknn.knn_bruteforce(x, k)
    u, v, w = oknn.knn_union_pairs(ref_i, ref_d, sigma)
    eu, ev, val = B.sc_knn_union_pairs(_dev(ref_i, torch.int32), _dev(ref_d, torch.float64), sigma)
    eu, ev, val = eu.cpu().numpy().astype(np.int64), ev.cpu().numpy().astype(np.int64), val.cpu().numpy()
    assert np.all(eu < ev)
    order = np.lexsort((ev, eu))                     # the library lists by emitting row; the set is what is unique
    np.testing.assert_array_equal(eu[order], u)
    np.testing.assert_array_equal(ev[order], v)
    np.testing.assert_allclose(val[order], w, rtol=1e-14, atol=0)


def test_union_pairs_skip_invalid_and_repeated_entries(B):
    # hand-made lists: -1 padding, a self reference, a neighbour listed twice, an out-of-range index
    idx = np.array([[1, 1, -1], [0, 2, 1], [7, 0, -1], [2, 3, 0]], dtype=np.int32)
    dist = np.array([[1.0, 1.0, 9.0], [1.0, 2.0, 0.0], [9.0, 3.0, 9.0], [4.0, 0.0, 5.0]])
    eu, ev, val = B.sc_knn_union_pairs(_dev(idx, torch.int32), _dev(dist, torch.float64), 0.0)
    got = sorted(zip(eu.cpu().tolist(), ev.cpu().tolist(), val.cpu().tolist()))
    # {0,1} from row 0; {1,2} from row 1; {0,2} from row 2 (row 0 does not list 2); {2,3} and {0,3} from row 3
    assert got == [(0, 1, 1.0), (0, 2, 3.0), (0, 3, 5.0), (1, 2, 2.0), (2, 3, 4.0)]


def test_points_to_graph_chain(B):
    """points -> sc_knn_search -> sc_knn_union_pairs (Gaussian weights) -> sc_coo_to_csr: the matrix equals the
    oracle's (dense, from its own neighbours and pairs), and the seeded input generator's graph of the same points."""
    from oracle import similarity as osim
    cfg = wl.CONFIGS[1]
    x, _ = wl.mixture_points(cfg)
    n = x.shape[0]
    ref_i, ref_d = oknn.knn_bruteforce(x, cfg.k_nn)
    sigma = float(np.median(ref_d))
    u, v, w = oknn.knn_union_pairs(ref_i, ref_d, sigma)
    dense = osim.coo_to_dense(u, v, w, n, True)
    idx, dist = B.sc_knn_search(_dev(x, torch.float64), cfg.k_nn)
    eu, ev, val = B.sc_knn_union_pairs(idx, dist, sigma)
    rp, co, va = B.sc_coo_to_csr(eu, ev, val, n, True)
    rp, co, va = rp.cpu().numpy(), co.cpu().numpy(), va.cpu().numpy()
    assert osim.csr_rows_sorted(rp, co)
    got = np.zeros((n, n))
    got[np.repeat(np.arange(n), np.diff(rp)), co] = va
    np.testing.assert_allclose(got, dense, rtol=1e-12, atol=0)
    assert np.count_nonzero(got) == rp[-1] == 2 * len(u)
    graph, gsigma = wl.knn_gaussian_graph(x, cfg.k_nn, "cpu")
    if graph[3] == n:                                  # the generator dropped no isolated point on this workload
        assert abs(gsigma - sigma) <= 1e-12 * sigma
        np.testing.assert_array_equal(rp, graph[0])
        np.testing.assert_array_equal(co, graph[1])
        np.testing.assert_allclose(va, graph[2], rtol=1e-6, atol=0)


def test_search_at_benchmark_size_on_sampled_queries(B):
    """Config 2's points (n = 100,000, d = 32, k_nn = 20): 48 sampled queries against the oracle's definition."""
    cfg = wl.CONFIGS[2]
    x, _ = wl.mixture_points(cfg)
    idx, dist = B.sc_knn_search(_dev(x, torch.float64), cfg.k_nn)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    rng = np.random.default_rng(5)
    ids = np.arange(x.shape[0])
    for i in rng.choice(x.shape[0], size=48, replace=False):
        diff = x - x[i]
        d2 = (diff * diff).sum(axis=1)
        d2[i] = np.inf
        order = np.lexsort((ids, d2))[:cfg.k_nn]
        np.testing.assert_array_equal(idx[i], order)
        np.testing.assert_allclose(dist[i], np.sqrt(d2[order]), rtol=1e-13)
    assert np.all(np.diff(dist, axis=1) >= 0) and idx.min() >= 0 and idx.max() < x.shape[0]


def _sampled(x, k, rows, idx, dist):
    """The lists of `rows` against the oracle's distances of those rows alone."""
    for i in rows:
        d2 = ((x - x[i]) ** 2).sum(axis=1)
        d2[i] = np.inf
        ref = np.lexsort((np.arange(x.shape[0]), d2))[:k]
        same = idx[i] == ref
        # two whose sums agree to the rounding of d + 2 additions may change places
        tol = (x.shape[1] + 2) * 2.3e-16
        assert np.all(np.abs(d2[idx[i]][~same] - d2[ref][~same]) <= 2 * tol * d2[ref][~same]), i
        np.testing.assert_allclose(dist[i], np.sqrt(d2[ref]), rtol=1e-13, atol=0)


# more queries than one round of the screen takes, the last round ragged; and with so many equal points among the rows of
# either round that the screen gives up on them
@pytest.mark.parametrize("kind", ["random", "equal at the start", "equal at the end"])
def test_screened_search_in_two_rounds(B, kind):
    n, d, k = 60_001, 8, 200                    # rounds of 55,296 queries: 256 MB of maxima and lists
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, d))
    if kind == "equal at the start":
        x[:900] = x[0]
    elif kind == "equal at the end":
        x[-900:] = x[-1]
    idx, dist = B.sc_knn_search(_dev(x, torch.float64), k)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    assert np.all(idx != np.arange(n)[:, None]) and np.all(np.diff(dist, axis=1) >= 0)
    cut = 55_296
    rows = np.concatenate([[0, 1, 898, 901, n - 1, n - 2, n - 901], np.arange(cut - 70, cut + 70, 7), rng.integers(0, n, 40)])
    _sampled(x, k, rows, idx, dist)


def test_search_without_room_for_the_screen(B):
    """290 MB of scratch for the screen, 160 MB there: the fp64 kernel alone gives the same lists."""
    n, d, k = 400_000, 4, 8
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    x = torch.randn((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    idx, dist = B.sc_knn_search(x, k)
    got = [torch.empty_like(idx), torch.empty_like(dist)]
    B.sc_release_cache()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    for _ in range(8):                          # what is reported as free comes down in steps
        more = torch.cuda.mem_get_info()[0] - (160 << 20)
        if more < 8 << 20:
            break
        held.append(torch.empty(more, dtype=torch.uint8, device="cuda:0"))
    code = B.lib().sc_knn_search(x.data_ptr(), d, n, d, k, got[0].data_ptr(), got[1].data_ptr(),
                                 torch.cuda.current_stream().cuda_stream)
    del held
    torch.cuda.empty_cache()
    assert code == B.SC_OK and torch.equal(got[0], idx) and torch.equal(got[1], dist)


# grouped points: cells with ragged last tiles, every padded dimension, clusters and none (then every pair is looked at),
# outliers in the cells, a common offset, equal points, more neighbours than a cell has points, two rounds of queries
@pytest.mark.parametrize("n,d,k,kind", [(62_000, 3, 10, "clusters"), (61_300, 16, 7, "clusters"), (45_001, 32, 20, "clusters"),
                                        (43_400, 17, 5, "random"), (31_007, 64, 32, "clusters"), (22_000, 100, 12, "clusters"),
                                        (63_000, 8, 200, "clusters"), (62_003, 2, 20, "outliers"), (45_000, 32, 6, "offset"),
                                        (62_500, 5, 9, "equal"), (61_999, 12, 3, "line")])
def test_grouped_search(B, n, d, k, kind, monkeypatch):
    rng = np.random.default_rng(3 * n + d)
    x = rng.standard_normal((n, d))
    if kind == "line":            # along a curve, in order
        t = np.linspace(0.0, 30.0, n)[:, None]
        x = np.sin(t * np.arange(1, d + 1) / d) * 5.0 + 1e-3 * x
    elif kind != "random":
        x += 15.0 * rng.standard_normal((90, d))[rng.integers(0, 90, n)]
    if kind == "outliers":
        x[::37] = 300.0 * rng.standard_normal((x[::37].shape[0], d))
    elif kind == "offset":
        x += 1e5
    elif kind == "equal":
        x[100:1100] = x[100]
    dx = _dev(x, torch.float64)
    before = B.sc_counter(B.SC_COUNTER_GROUPED_SEARCHES)
    idx, dist = B.sc_knn_search(dx, k)
    assert B.sc_counter(B.SC_COUNTER_GROUPED_SEARCHES) - before == (0 if kind == "random" else 1)
    # every list of every point, as without the groups
    monkeypatch.setenv("SCEIG_NO_GROUPS", "1")
    plain_idx, plain_dist = B.sc_knn_search(dx, k)
    assert B.sc_counter(B.SC_COUNTER_GROUPED_SEARCHES) - before <= 1
    assert torch.equal(idx, plain_idx) and torch.equal(dist, plain_dist)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    assert np.all(idx != np.arange(n)[:, None]) and np.all(np.diff(dist, axis=1) >= 0) and idx.min() >= 0
    _sampled(x, k, np.concatenate([[0, 99, 100, 600, n - 1], rng.integers(0, n, 120)]), idx, dist)


# many neighbours in few tiles: the lists of candidates of some queries run over
@pytest.mark.parametrize("n,d,k,kind", [(62_001, 2, 50, "normal"), (100_003, 2, 50, "normal"), (100_000, 3, 100, "uniform"),
                                        (62_000, 10, 100, "tight"), (30_011, 70, 60, "tight"), (62_500, 2, 200, "uniform"), (62_000, 16, 60, "line")])
def test_grouped_search_whose_lists_run_over(B, n, d, k, kind, monkeypatch):
    gen = torch.Generator(device="cuda:0").manual_seed(n + d)
    x = torch.randn((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    if kind == "uniform":
        x = torch.rand((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    elif kind == "line":              # closer to one another than the screen can tell: nearly all run over
        x = 0.01 * x + torch.linspace(0, 50, n, dtype=torch.float64, device="cuda:0")[:, None]
    elif kind == "tight":             # clusters of very different widths
        at = torch.arange(n, device="cuda:0") % 40
        x = x * (10.0 ** (-2.0 * torch.rand(40, dtype=torch.float64, device="cuda:0", generator=gen)))[at, None]
        x += 8.0 * torch.randn((40, d), dtype=torch.float64, device="cuda:0", generator=gen)[at]
    fp64 = B.sc_counter(B.SC_COUNTER_FP64_SEARCHES)
    idx, dist = B.sc_knn_search(x, k)
    # clusters a hundredth as wide as the points are far apart: the screen cannot tell their points apart
    assert kind in ("tight", "line") or B.sc_counter(B.SC_COUNTER_FP64_SEARCHES) == fp64
    monkeypatch.setenv("SCEIG_NO_GROUPS", "1")
    plain_idx, plain_dist = B.sc_knn_search(x, k)
    assert torch.equal(idx, plain_idx) and torch.equal(dist, plain_dist)


@pytest.mark.parametrize("n,d,kind,grouped", [(90_000, 4, "normal", 0), (66_000, 5, "curve", 0), (66_000, 8, "curve", 0),
                                              (66_000, 6, "uniform", 0), (62_000, 3, "normal", 0), (66_000, 3, "uniform", 1), (66_000, 2, "normal", 1),
                                              (66_000, 10, "blobs", 1), (45_000, 32, "blobs", 1), (45_000, 32, "normal", 0)])
def test_points_are_grouped_where_it_pays(B, n, d, kind, grouped):
    """Without clusters in four dimensions and more the lists of the groups keep a third of the pairs and more, at several times
    the cost of a pair: such points are searched as they are (90,000 normal ones of 4 coordinates took 1.8 times as long)."""
    gen = torch.Generator(device="cuda:0").manual_seed(d)
    x = torch.randn((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    if kind == "uniform":
        x = torch.rand((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    elif kind == "curve":         # three parameters, bent
        t = 6.0 * torch.rand((n, 3), dtype=torch.float64, device="cuda:0", generator=gen)
        x = torch.sin(t @ torch.randn((3, d), dtype=torch.float64, device="cuda:0", generator=gen)) + 0.05 * x
    elif kind == "blobs":
        x += 8.0 * torch.randn((60, d), dtype=torch.float64, device="cuda:0", generator=gen)[torch.arange(n, device="cuda:0") % 60]
    before = B.sc_counter(B.SC_COUNTER_GROUPED_SEARCHES)
    B.sc_knn_search(x, 10)
    assert B.sc_counter(B.SC_COUNTER_GROUPED_SEARCHES) - before == grouped
