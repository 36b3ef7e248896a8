"""GPU parity of the k-means step (Section IV-C, Algorithms 4 and 5) against the oracle, through the C ABI.

Labels and chosen seeds are integers decided by fp64 arithmetic: both sides decide in fp64, the kernel on the expanded
form |c|^2 - 2<v,c> and the oracle on the direct sum of squared differences.  The two may differ only where two
candidates are equal to rounding, so: every label / seed must be the oracle's, or a candidate that the oracle's own
numbers cannot tell from its choice (checked, and such points must be rare); centres agree to 1e-11 relative."""
import numpy as np
import pytest

from oracle import kmeans as okm
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


def _blobs(n, d, k, seed, spread=0.15):
    return wl.gaussian_blobs(n, d, k, seed, spread)


def _embedding_like(n, k, seed):
    return wl.embedding_like(n, k, seed)


def _dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda:0")


def _check_labels(x, cen_used, labels_gpu, labels_ref, dist_ref, max_ambiguous):
    """labels_gpu equals labels_ref except where the oracle's distances to the two labels agree to rounding."""
    diff = np.flatnonzero(labels_gpu != labels_ref)
    scale = float((x * x).sum(axis=1).max() + (cen_used * cen_used).sum(axis=1).max())
    for i in diff:
        assert abs(dist_ref[i, labels_gpu[i]] - dist_ref[i, labels_ref[i]]) <= 1e-12 * scale, (i, dist_ref[i])
    assert diff.size <= max_ambiguous, diff.size


CASES = [
    # n, d, k: several 64-row tiles / 64-centre tiles with ragged tails, d not a multiple of 4, k = 1, k = n
    ("blobs", 5003, 7, 5),
    ("blobs", 12345, 33, 70),
    ("blobs", 4097, 130, 257),
    ("embed", 20011, 100, 100),
    ("blobs", 300, 3, 1),
    ("blobs", 64, 2, 64),
    ("uniform", 6000, 6, 40),
]


def _points(kind, n, d, k, seed):
    if kind == "blobs":
        return _blobs(n, d, max(k, 1), seed)
    if kind == "embed":
        return _embedding_like(n, k, seed)
    return np.random.default_rng(seed).uniform(-1, 1, size=(n, d))


@pytest.mark.parametrize("kind,n,d,k", CASES)
def test_kmeanspp_matches_oracle(B, kind, n, d, k):
    x = _points(kind, n, d, k, seed=n + k)
    for seed in (1, 2):
        ref = okm.kmeanspp_indices(x, k, seed)
        chosen, cen = B.sc_kmeanspp(_dev(x), k, seed)
        got = chosen.cpu().numpy().astype(np.int64)
        if not np.array_equal(got, ref):
            # a draw may land within rounding of a boundary of the prefix sums: then the neighbouring point is as valid
            first = int(np.flatnonzero(got != ref)[0])
            assert first > 0
            d2 = okm.sq_distances_to(x, x[ref[0]])
            for j in ref[1:first]:
                d2 = np.minimum(d2, okm.sq_distances_to(x, x[j]))
            cs = np.cumsum(d2)
            r = okm.uniform01(seed, first) * cs[-1]
            lo, hi = sorted((int(got[first]), int(ref[first])))
            assert np.all(np.abs(cs[lo:hi] - r) <= 1e-12 * cs[-1]), (first, got[first], ref[first])
            pytest.skip("draw within rounding of a prefix-sum boundary; later draws legitimately differ")
        np.testing.assert_array_equal(cen.cpu().numpy(), x[ref])


@pytest.mark.parametrize("colmajor", [False, True])
@pytest.mark.parametrize("kind,n,d,k", CASES)
def test_lloyd_matches_oracle(B, kind, n, d, k, colmajor):
    x = _points(kind, n, d, k, seed=7 * n + k)
    init = x[okm.kmeanspp_indices(x, k, 3)]
    labels_ref, cen_ref, iters_ref, hist_ref, conv_ref = okm.lloyd(x, init, 60)
    pts = _dev(x.T) if colmajor else _dev(x)
    labels, cen, code, st = B.sc_kmeans_lloyd(pts, _dev(init), 60, colmajor=colmajor)
    lg = labels.cpu().numpy().astype(np.int64)
    # the labels of the last step were computed from the centres before the (skipped or last) update
    _, dist_ref = okm.assign(x, cen_ref if conv_ref else init)
    if conv_ref:
        _check_labels(x, cen_ref, lg, labels_ref, dist_ref, max_ambiguous=max(2, n // 2000))
        assert st["iterations"] == iters_ref and st["converged"] == 1 and code == 0
        np.testing.assert_allclose(cen.cpu().numpy(), cen_ref, rtol=1e-11, atol=1e-12)
        assert abs(st["objective"] - hist_ref[-1]) <= 1e-9 * max(1.0, hist_ref[-1])
    else:
        assert code == 1 and st["converged"] == 0 and st["iterations"] == 60
    assert lg.min() >= 0 and lg.max() < k


def test_one_lloyd_step_element_by_element(B):
    """One labelling step + one update from fixed centres: no iteration, so every label and centre is comparable."""
    n, d, k = 7001, 19, 37
    x = _blobs(n, d, k, 5, spread=0.6)
    init = x[np.random.default_rng(1).choice(n, k, replace=False)].copy()
    init[5] = 100.0  # a centre that attracts nobody keeps its place
    labels_ref, dist_ref = okm.assign(x, init)
    cen_ref = okm.update_centroids(x, labels_ref, init)
    labels, cen, code, st = B.sc_kmeans_lloyd(_dev(x), _dev(init), 1)
    assert code == 1 and st["iterations"] == 1 and st["last_changes"] == n
    _check_labels(x, init, labels.cpu().numpy().astype(np.int64), labels_ref, dist_ref, max_ambiguous=0)
    np.testing.assert_allclose(cen.cpu().numpy(), cen_ref, rtol=1e-12, atol=1e-13)
    np.testing.assert_array_equal(cen.cpu().numpy()[5], init[5])


def test_kmeans_whole_and_bitwise_repeatable(B):
    n, d, k = 30011, 24, 24
    x = _embedding_like(n, k, 9)
    labels_ref, cen_ref, iters_ref, hist_ref, conv_ref = okm.kmeans(x, k, 42, 100)
    assert conv_ref
    out = [B.sc_kmeans(_dev(x), k, 42, 100) for _ in range(2)]
    (l0, c0, code0, st0), (l1, c1, _, _) = out
    assert torch.equal(l0, l1) and torch.equal(c0, c1)
    assert code0 == 0 and st0["iterations"] == iters_ref
    np.testing.assert_array_equal(l0.cpu().numpy(), labels_ref)
    np.testing.assert_allclose(c0.cpu().numpy(), cen_ref, rtol=1e-11, atol=1e-12)


def test_kmeans_on_eigensolver_output(B):
    """Steps 3 and 4 of Section II chained on the device: row-normalised eigenvectors of a graph with 6 components
    are clustered into exactly those components."""
    from oracle import components as ocomp
    from paper_1802_04450_amd import workloads as wl
    cfg = wl.reduced(wl.CONFIGS[2], n=6007, components=6, k=6)
    (rp, c, v, n), _, _ = wl.build_config_graph(cfg, device="cpu")
    drp, dc, dv = B.csr_to_device(rp, c, v)
    evals, evecs, code, _ = B.sc_laplacian_eigsh(drp, dc, dv, 6, 1e-10, flags=B.SC_FLAG_ROW_NORMALIZE)
    assert code == 0
    labels, cen, kcode, st = B.sc_kmeans(evecs, 6, 5, 100, colmajor=True)
    ncomp, comp = ocomp.component_labels(rp, c, v)
    assert ncomp == 6 and kcode == 0
    lg = labels.cpu().numpy()
    # Points of one component share their embedding row (to the solver's tolerance), so squared-distance sampling
    # draws every seed from a component that has none yet, and the clustering is the component partition up to the
    # names of the clusters.
    pairs = {(int(a), int(b)) for a, b in zip(comp, lg)}
    assert len(pairs) == 6 and len({p[0] for p in pairs}) == 6 and len({p[1] for p in pairs}) == 6
    assert st["objective"] <= 1e-12 * n


def test_kmeans_argument_errors(B):
    x = _dev(np.zeros((10, 3)))
    lib = B.lib()
    out_l = torch.empty(10, dtype=torch.int32, device="cuda:0")
    out_c = torch.empty((4, 3), dtype=torch.float64, device="cuda:0")
    assert lib.sc_kmeans(x.data_ptr(), 3, 0, 10, 3, 11, 0, 10, out_l.data_ptr(), out_c.data_ptr(), None, None) == B.SC_EDOMAIN
    assert lib.sc_kmeans(x.data_ptr(), 3, 0, 10, 3, 0, 0, 10, out_l.data_ptr(), out_c.data_ptr(), None, None) == B.SC_EDOMAIN
    assert lib.sc_kmeans(x.data_ptr(), 2, 0, 10, 3, 4, 0, 10, out_l.data_ptr(), out_c.data_ptr(), None, None) == B.SC_EDOMAIN
    assert lib.sc_kmeans(None, 3, 0, 10, 3, 4, 0, 10, out_l.data_ptr(), out_c.data_ptr(), None, None) == B.SC_EINVAL
    assert lib.sc_kmeans(x.data_ptr(), 3, 0, 10, 3, 4, 0, 0, out_l.data_ptr(), out_c.data_ptr(), None, None) == B.SC_EDOMAIN
    assert lib.sc_kmeans_lloyd(x.data_ptr(), 3, 0, 10, 3, 4, None, 5, out_l.data_ptr(), None, None) == B.SC_EINVAL


# the counting sort of the update at the edges of its blocks and of its range of clusters, and the radix sort beyond
# and the labelling in parts of the centres on both sides of where it begins, with a last part that is not full
@pytest.mark.parametrize("n,d,k", [(2000, 10, 448), (2000, 10, 449), (5000, 130, 257), (1000, 300, 161), (32704, 20, 520),
                                   (32705, 20, 520), (520, 7, 513), (70, 2, 70), (1023, 1, 1), (1024, 2, 64), (1025, 5, 3), (4500, 9, 1024), (4500, 3, 1025), (3000, 129, 200)])
def test_update_over_its_ranges(B, n, d, k):
    rng = np.random.default_rng(n + d + k)
    x = rng.standard_normal((n, d))
    init = x[rng.choice(n, k, replace=False)].copy()
    labels_ref, dist_ref = okm.assign(x, init)
    cen_ref = okm.update_centroids(x, labels_ref, init)
    labels, cen, _, _ = B.sc_kmeans_lloyd(_dev(x), _dev(init), 1)
    lg = labels.cpu().numpy().astype(np.int64)
    _check_labels(x, init, lg, labels_ref, dist_ref, max_ambiguous=2)
    same = np.ones(k, dtype=bool)      # centres of clusters that the ambiguous points moved between are not comparable
    same[np.concatenate([lg[lg != labels_ref], labels_ref[lg != labels_ref]])] = False
    # sums of at most n numbers below 6 in another order: n 2^-53 of the sum of the moduli
    np.testing.assert_allclose(cen.cpu().numpy()[same], cen_ref[same], rtol=0, atol=6.0 * n * 2.0 ** -53)


# the seeding with the bf16 copy of the points: with and without its own draw, a common offset, equal points, coordinates
# whose squares leave the range of a float at either end, or of which no scale is made
@pytest.mark.parametrize("n,d,k,kind", [(62501, 64, 33, "blobs"), (120003, 34, 40, "blobs"), (45001, 90, 32, "offset"),
                                        (40001, 101, 35, "equal"), (62501, 64, 40, 1e20), (62501, 64, 40, 1e19),
                                        (120003, 34, 40, 1e25), (62501, 64, 40, 3e-23), (62501, 64, 40, 1e-21),
                                        (62501, 64, 40, 1e-30), (62501, 64, 33, 1e120), (62501, 64, 33, "two scales"),
                                        # around the numbers of blocks from which two go to a workgroup and the draw moves
                                        # out, an odd number of them, a last block of one point; the most coordinates
                                        (65409, 105, 32, "blobs"), (65473, 112, 33, "blobs"), (65537, 113, 32, "blobs"),
                                        (115137, 40, 32, "offset"), (115201, 40, 34, "equal"), (65600, 64, 33, 1e20),
                                        # few and many coordinates: one to several batches of a row's loads
                                        (270_001, 16, 32, "blobs"), (250_003, 17, 33, "offset"), (130_001, 31, 32, "equal"),
                                        (31_000, 130, 32, "blobs"), (9_001, 500, 33, "offset")])
def test_screened_seeding_equals_plain_distances(B, n, d, k, kind):
    x = _blobs(n, d, 25, seed=n, spread=0.3)
    if kind == "offset":
        x += 1e7
    elif kind == "equal":
        x[1:] = x[0] + np.repeat(np.arange(1.0, n)[:, None] % 7, d, axis=1)
    elif kind == "two scales":       # one point far away: the others' squares are near the smallest float after scaling
        x[1:] *= 1e-20
    elif isinstance(kind, float):
        x *= kind
    chosen = B.sc_kmeanspp(_dev(x), k, 5)[0].cpu().numpy().astype(np.int64)
    # draw by draw from the chosen points themselves: the index must be where the prefix sum passes u * total, to the
    # rounding of sums of n numbers
    d2 = okm.sq_distances_to(x, x[chosen[0]])
    for i in range(1, k):
        cs = np.cumsum(d2)
        r = okm.uniform01(5, i) * cs[-1]
        tol = 4.0 * n * 2.0 ** -53 * cs[-1]
        j = chosen[i]
        assert (j == n - 1 or cs[j] > r - tol) and (j == 0 or cs[j - 1] <= r + tol), (i, j)
        d2 = np.minimum(d2, okm.sq_distances_to(x, x[j]))


def test_points_without_a_finite_distance_break_nothing(B):
    x = _blobs(5000, 20, 6, seed=3)
    bad = np.array([17, 2048, 4999])
    x[bad[0], 3], x[bad[1], 7], x[bad[2], 0] = np.nan, np.inf, -np.inf
    init = np.delete(x, bad, axis=0)[:6].copy()
    labels, cen, _, _ = B.sc_kmeans_lloyd(_dev(x), _dev(init), 1)
    good = np.delete(np.arange(5000), bad)
    labels_ref, _ = okm.assign(x[good], init)
    np.testing.assert_array_equal(labels.cpu().numpy()[good], labels_ref)


def test_a_converging_run_with_points_without_a_finite_distance(B):
    """Points with a NaN coordinate have no label, move no centre and leave no objective; the rest is clustered as if they
    were not there."""
    x = _blobs(5000, 20, 6, seed=3)
    bad = np.array([0, 17, 2048, 4999])
    x[bad, [0, 3, 7, 19]] = np.nan
    good = np.delete(np.arange(5000), bad)
    init = x[good][okm.kmeanspp_indices(x[good], 6, 1)].copy()
    labels_ref, cen_ref, iters_ref, _, conv_ref = okm.lloyd(x[good], init, 60)
    assert conv_ref
    labels, cen, code, st = B.sc_kmeans_lloyd(_dev(x), _dev(init), 60)
    assert code == 0 and st["converged"] == 1 and st["iterations"] == iters_ref and np.isnan(st["objective"])
    lg = labels.cpu().numpy()
    np.testing.assert_array_equal(lg[good], labels_ref)
    assert np.all(lg[bad] == 2 ** 31 - 1)
    np.testing.assert_allclose(cen.cpu().numpy(), cen_ref, rtol=1e-11, atol=1e-12)


# both ways of grouping the points, with numbers of clusters on both sides of a power of two
@pytest.mark.parametrize("k", [512, 1023, 1024, 1025, 2047, 2048, 2049, 4096])
def test_points_without_a_label_belong_to_no_cluster(B, k):
    n, d = 9000, 5
    x = _blobs(n, d, 30, seed=k, spread=0.5)
    bad = np.array([0, 17, 2048, 4095, 8999])
    good = np.delete(np.arange(n), bad)
    init = x[good][np.random.default_rng(k).choice(good.size, k, replace=False)].copy()
    x[bad, 2] = np.nan
    labels_ref, _ = okm.assign(x[good], init)
    cen_ref = okm.update_centroids(x[good], labels_ref, init)
    labels, cen, _, _ = B.sc_kmeans_lloyd(_dev(x), _dev(init), 1)
    lg = labels.cpu().numpy()
    assert np.all(lg[bad] == 2 ** 31 - 1)
    np.testing.assert_array_equal(lg[good], labels_ref)
    np.testing.assert_allclose(cen.cpu().numpy(), cen_ref, rtol=0, atol=6.0 * n * 2.0 ** -53)


def test_seeding_without_room_for_its_copy(B):
    """512 MB of points are staged, and of the 150 MB that the seeding would like 88 MB are there."""
    n, d, k = 1_000_000, 64, 40
    gen = torch.Generator(device="cuda:0").manual_seed(7)
    x = torch.randn((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    chosen, cen = B.sc_kmeanspp(x, k, 3)
    got = [torch.empty_like(chosen), torch.empty_like(cen)]
    B.sc_release_cache()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    for _ in range(8):                          # what is reported as free comes down in steps
        more = torch.cuda.mem_get_info()[0] - n * d * 8 - (88 << 20)
        if more < 8 << 20:
            break
        held.append(torch.empty(more, dtype=torch.uint8, device="cuda:0"))
    code = B.lib().sc_kmeanspp(x.data_ptr(), d, 0, n, d, k, 3, got[0].data_ptr(), got[1].data_ptr(),
                               torch.cuda.current_stream().cuda_stream)
    del held
    torch.cuda.empty_cache()
    assert code == B.SC_OK and torch.equal(got[0], chosen) and torch.equal(got[1], cen)


def test_labelling_in_parts_takes_the_lowest_index_on_ties(B):
    """Equal centres in different parts of the centres: the first of them gets the points."""
    rng = np.random.default_rng(8)
    n, d, k = 700, 12, 700
    x = rng.integers(-4, 5, size=(n, d)).astype(np.float64)       # all products exact
    init = x[rng.permutation(n)].copy()
    init[600:] = init[:100]
    init[64:128] = init[:64]
    labels_ref, _ = okm.assign(x, init)
    labels, _, _, _ = B.sc_kmeans_lloyd(_dev(x), _dev(init), 1)
    np.testing.assert_array_equal(labels.cpu().numpy(), labels_ref)


# the screened labelling: ragged tiles of points and of centres, one to all pieces of 16 coordinates, the wide form, centres in
# more than one chunk of LDS, blobs with several centres each, data far from the origin, equal points, a NaN
@pytest.mark.parametrize("n,d,k,kind", [(500_003, 5, 161, "blobs"), (262_147, 16, 97, "blobs"), (100_001, 33, 130, "blobs"),
                                        (40_010, 100, 100, "split"), (33_333, 128, 101, "blobs"), (30_001, 129, 104, "blobs"),
                                        (13_007, 300, 110, "split"), (200_001, 20, 100, "offset"), (60_000, 70, 96, "equal"),
                                        (60_001, 70, 96, "nan"), (2_100, 130, 1500, "blobs")])
def test_screened_labelling_is_the_nearest_centre(B, n, d, k, kind, monkeypatch):
    gen = torch.Generator(device="cuda:0").manual_seed(n + d)
    blobs = k // 4 if kind == "split" else k
    cen = torch.randn((blobs, d), dtype=torch.float64, device="cuda:0", generator=gen)
    x = cen[torch.randint(0, blobs, (n,), device="cuda:0", generator=gen)]
    x = x + 0.2 * torch.randn((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    if kind == "offset":
        x += 1e5
    elif kind == "equal":
        x[: n // 2] = x[0]
    elif kind == "nan":
        x[17, 3] = float("nan")
    init = x[torch.randperm(n - 100, device="cuda:0", generator=gen)[:k] + 100].clone()
    if kind == "equal":
        init[1] = init[0]
    monkeypatch.setenv("SCEIG_FORCE_LABEL_SCREEN", "1")       # three steps do not bring in its cost in all of these
    seen = B.sc_counter(B.SC_COUNTER_SCREENED_LABELLINGS)
    labels, centres, code, stats = B.sc_kmeans_lloyd(x, init, 3)
    # no scale with a NaN; half of the points as near to two equal centres: the screen is given up after the first step
    by_screen = 0 if kind in ("equal", "nan") else stats["iterations"]
    assert B.sc_counter(B.SC_COUNTER_SCREENED_LABELLINGS) - seen == by_screen
    # the same labels and centres as by the fp64 labelling alone
    with monkeypatch.context() as m:
        m.setenv("SCEIG_NO_LABEL_SCREEN", "1")
        plain_labels, plain_centres, _, _ = B.sc_kmeans_lloyd(x, init, 3)
    assert B.sc_counter(B.SC_COUNTER_SCREENED_LABELLINGS) - seen == by_screen
    assert torch.equal(labels, plain_labels)
    assert torch.equal(torch.nan_to_num(centres), torch.nan_to_num(plain_centres))
    # the labels are those of the last labelling step: its centres come out of a run one update shorter
    _, before, _, st2 = B.sc_kmeans_lloyd(x, init, 2)
    assert stats["iterations"] == 3 or stats["converged"]
    cen_used = before if stats["iterations"] == 3 else centres
    for r0 in range(0, n, 8192):
        xr = x[r0:r0 + 8192]
        v = (cen_used * cen_used).sum(1)[None, :] - 2.0 * (xr @ cen_used.T)
        lab = labels[r0:r0 + 8192].long()
        fine = torch.isfinite(v).all(1)
        got = torch.gather(v, 1, lab.clamp(0, k - 1)[:, None])[:, 0]
        # the label's value is the smallest, up to what the fp64 sums of either side are off by
        size = (xr.norm(dim=1) + cen_used.norm(dim=1).max()) ** 2
        assert bool((got - v.min(1)[0] <= (4 * d + 16) * 1.2e-16 * size)[fine].all()), r0
        assert bool(((lab >= 0) & (lab < k))[fine].all())


# the seeding and the labelling both by their reduced copies, which share the points' mean and scale: the same as without the
# labelling's, and as steps of their own from the chosen points, which make them again
@pytest.mark.parametrize("n,d,k,kind", [(40_003, 100, 101, "normal"), (125_003, 33, 97, "offset"), (125_000, 32, 100, "small")])
def test_mean_and_scale_shared_by_seeding_and_labelling(B, n, d, k, kind, monkeypatch):
    gen = torch.Generator(device="cuda:0").manual_seed(n + k)
    x = torch.randn((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    x = 300.0 + x if kind == "offset" else 1e-9 * x if kind == "small" else x
    monkeypatch.setenv("SCEIG_FORCE_LABEL_SCREEN", "1")
    seen = B.sc_counter(B.SC_COUNTER_SCREENED_LABELLINGS)
    labels, centres = B.sc_kmeans(x, k, 5, max_iter=4)[:2]
    assert B.sc_counter(B.SC_COUNTER_SCREENED_LABELLINGS) > seen
    alone_labels, alone_centres = B.sc_kmeans_lloyd(x, B.sc_kmeanspp(x, k, 5)[1], 4)[:2]
    assert torch.equal(labels, alone_labels) and torch.equal(centres, alone_centres)
    monkeypatch.setenv("SCEIG_NO_LABEL_SCREEN", "1")
    plain_labels, plain_centres = B.sc_kmeans(x, k, 5, max_iter=4)[:2]
    assert torch.equal(labels, plain_labels) and torch.equal(centres, plain_centres)


# Draws in one launch.  Without the screen: 16 draws and blocks of points from one to the 256 that it is taken for; with it: one and
# several blocks a workgroup, the last ones ragged, up to the blocks that it takes (1,800) and the LDS (128 coordinates there)
@pytest.mark.parametrize("n,d,k,data,one", [(16, 3, 16, "blobs", True), (65, 1, 16, "blobs", True), (4097, 17, 31, "blobs", True),
                                            (16384, 5, 16, "blobs", True), (16385, 5, 16, "blobs", False), (500, 7, 15, "blobs", False),
                                            (2000, 130, 20, "blobs", True), (3000, 9, 40, "few", True), (700, 4, 20, "nan", True),
                                            (40_000, 100, 33, "blobs", True), (115_200, 35, 40, "blobs", True),
                                            (115_201, 35, 40, "blobs", False), (115_200, 128, 34, "blobs", True),
                                            (100_003, 99, 32, "blobs", True), (60_000, 67, 32, "embedding", True),
                                            (50_000, 80, 32, "few", True), (50_000, 80, 32, "huge", True), (50_000, 80, 32, "nan", True)])
def test_draws_in_one_launch(B, monkeypatch, n, d, k, data, one):
    """The points drawn by one launch, by a launch a draw, and when the one launch finds that its workgroups cannot all have
    started: the same, also where there are fewer different points than draws, no scale for the screen, or no number."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d)
    cen = torch.randn((k, d), dtype=torch.float64, generator=g, device="cuda")
    lab = torch.randint(0, k, (n,), generator=g, device="cuda")
    spread = {"embedding": 1e-6, "few": 0.0}.get(data, 0.15)
    x = (cen[lab[:]] if data != "few" else cen[lab % 7]) + spread * torch.randn((n, d), dtype=torch.float64, generator=g, device="cuda")
    if data == "huge":
        x *= 1e140
    if data == "nan":
        x[n // 2, d // 2] = float("nan")
    picked = []
    for env in ({}, {"SCEIG_NO_FUSED": "1"}, {"SCEIG_FUSED_POLLS": "-1"}):
        for name, value in env.items():
            monkeypatch.setenv(name, value)
        before = B.sc_counter(B.SC_COUNTER_FUSED_SEEDINGS)
        chosen, out = B.sc_kmeanspp(x, k, 5)
        assert B.sc_counter(B.SC_COUNTER_FUSED_SEEDINGS) - before == (1 if one and not env else 0)
        for name in env:
            monkeypatch.delenv(name)
        picked.append(chosen)
        same = out == x[chosen.long()]
        assert bool((same | (out.isnan() & x[chosen.long()].isnan())).all())
    assert torch.equal(picked[0], picked[1]) and torch.equal(picked[2], picked[1])


# What is enqueued behind the one launch before the host knows whether its workgroups have all started: the rows of the points
# chosen.  The places of the points not drawn hold what was in the caller's memory, here numbers that are no point's.
@pytest.mark.parametrize("n,d,k", [(2000, 16, 32), (16, 3, 16), (45_000, 100, 40), (115_200, 128, 34)])
def test_draws_that_do_not_start_leave_points_chosen(B, monkeypatch, n, d, k):
    x = _dev(wl.gaussian_blobs(n, d, min(k, 10), 3, 0.3))
    chosen, centres = B.sc_kmeanspp(x, k, 5)
    torch.cuda.synchronize()
    monkeypatch.setenv("SCEIG_FUSED_POLLS", "-1")
    again = torch.full((k,), 0x7ffffff0, dtype=torch.int32, device="cuda:0")
    rows = torch.zeros((k, d), dtype=torch.float64, device="cuda:0")
    before = B.sc_counter(B.SC_COUNTER_FUSED_SEEDINGS)
    torch.cuda.synchronize()
    assert B.lib().sc_kmeanspp(x.data_ptr(), d, 0, n, d, k, 5, again.data_ptr(), rows.data_ptr(), 0) == B.SC_OK
    assert B.sc_counter(B.SC_COUNTER_FUSED_SEEDINGS) == before
    assert torch.equal(again, chosen) and torch.equal(rows, centres)


# two callers with streams of their own, and nothing that makes a call wait before its end (no statistics): the iterations' blocks
# of the one are free for the other only once its launches are done.  Up to 1,024 clusters and more of them (radix sort); calls
# that converge, after two labellings and after many, and calls that end at max_iter
@pytest.mark.parametrize("n,d,k,max_iter,spread", [(3000, 4, 8, 50, 0.02), (20_000, 8, 64, 60, 0.6), (20_000, 8, 64, 3, 0.6),
                                                   (12_000, 4, 1100, 40, 0.3), (12_000, 4, 1100, 2, 0.3)])
def test_two_callers_at_once_without_statistics(B, n, d, k, max_iter, spread):
    import threading
    sets = [_dev(wl.gaussian_blobs(n, d, min(k, 40), seed, spread)) for seed in (1, 2)]
    alone = []
    for x in sets:
        labels, centres, code, _ = B.sc_kmeans(x, k, 9, max_iter=max_iter)
        assert code in (B.SC_OK, B.SC_NOT_CONVERGED)
        alone.append((labels, centres, code))
    rounds = 12
    labels = [[torch.full((n,), -7, dtype=torch.int32, device="cuda:0") for _ in range(rounds)] for _ in sets]
    centres = [[torch.zeros((k, d), dtype=torch.float64, device="cuda:0") for _ in range(rounds)] for _ in sets]
    codes = [[], []]
    torch.cuda.synchronize()

    def call(t):
        stream = torch.cuda.Stream()
        for r in range(rounds):
            codes[t].append(B.lib().sc_kmeans(sets[t].data_ptr(), d, 0, n, d, k, 9, max_iter, labels[t][r].data_ptr(),
                                              centres[t][r].data_ptr(), None, stream.cuda_stream))

    callers = [threading.Thread(target=call, args=(t,)) for t in range(2)]
    for c in callers:
        c.start()
    for c in callers:
        c.join()
    for t in range(2):
        for r in range(rounds):
            assert codes[t][r] == alone[t][2], (t, r)
            assert torch.equal(labels[t][r], alone[t][0]) and torch.equal(centres[t][r], alone[t][1]), (t, r)
