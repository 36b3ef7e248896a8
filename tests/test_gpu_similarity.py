"""GPU parity of the similarity-graph step (Section IV-A, Algorithm 1; Algorithm 2 step 4) against the oracle,
through the C ABI, and the chain points -> similarity -> CSR -> eigensolver input."""
import ctypes
import time

import numpy as np
import pytest

from oracle import similarity as osim
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


def _edges(n, ne, seed):
    rng = np.random.default_rng(seed)
    u = rng.integers(0, n, size=ne)
    v = rng.integers(0, n, size=ne)
    return u, v


@pytest.mark.parametrize("n,d,ne", [(5003, 90, 40011), (1000, 3, 7777), (300, 1, 500), (2000, 33, 20000),
                                    (700, 257, 3000), (10, 16, 0)])
@pytest.mark.parametrize("measure", [0, 1, 2])
def test_edge_similarity_matches_oracle(B, n, d, ne, measure):
    rng = np.random.default_rng(n + d + measure)
    x = rng.normal(size=(n, d)) + 2.0 * rng.normal(size=(n, 1))
    u, v = _edges(n, ne, 3)
    sigma = 1.7 * np.sqrt(d)
    if d == 1 and measure == 0:
        # one coordinate: every centred row is zero and the measure is 0/0 by its definition - NaN on both sides
        got = B.sc_edge_similarity(_dev(x, torch.float64), _dev(u, torch.int32), _dev(v, torch.int32), measure, sigma)
        with np.errstate(invalid="ignore", divide="ignore"):
            ref = osim.edge_similarity(x, u, v, measure, sigma)
        assert np.all(np.isnan(ref)) and bool(torch.all(torch.isnan(got)))
        return
    ref = osim.edge_similarity(x, u, v, measure, sigma) if ne else np.zeros(0)
    got = B.sc_edge_similarity(_dev(x, torch.float64), _dev(u, torch.int32), _dev(v, torch.int32), measure, sigma)
    np.testing.assert_allclose(got.cpu().numpy(), ref, rtol=1e-12, atol=1e-14)


def test_edge_similarity_strided_rows_and_errors(B):
    rng = np.random.default_rng(1)
    n, d = 400, 7
    big = torch.as_tensor(rng.normal(size=(n, 11)), device="cuda:0")        # odd leading dimension: scalar loads
    x = big[:, :d]
    u, v = _edges(n, 3000, 5)
    du, dv = _dev(u, torch.int32), _dev(v, torch.int32)
    val = torch.empty(3000, dtype=torch.float64, device="cuda:0")
    lib = B.lib()
    st = torch.cuda.current_stream().cuda_stream
    assert lib.sc_edge_similarity(x.data_ptr(), 11, n, d, du.data_ptr(), dv.data_ptr(), 3000, 0, 1.0, val.data_ptr(), st) == 0
    ref = osim.edge_similarity(big.cpu().numpy()[:, :d], u, v, 0)
    np.testing.assert_allclose(val.cpu().numpy(), ref, rtol=1e-12, atol=1e-14)
    assert lib.sc_edge_similarity(x.data_ptr(), 5, n, d, du.data_ptr(), dv.data_ptr(), 3000, 0, 1.0, val.data_ptr(), st) == B.SC_EDOMAIN
    assert lib.sc_edge_similarity(x.data_ptr(), 11, n, d, du.data_ptr(), dv.data_ptr(), 3000, 2, 0.0, val.data_ptr(), st) == B.SC_EDOMAIN
    assert lib.sc_edge_similarity(x.data_ptr(), 11, n, d, du.data_ptr(), dv.data_ptr(), 3000, 3, 1.0, val.data_ptr(), st) == B.SC_EDOMAIN
    assert lib.sc_edge_similarity(None, 11, n, d, du.data_ptr(), dv.data_ptr(), 3000, 0, 1.0, val.data_ptr(), st) == B.SC_EINVAL
    u2 = u.copy()
    u2[17] = n          # an index past the end is reported, not read
    assert lib.sc_edge_similarity(x.data_ptr(), 11, n, d, _dev(u2, torch.int32).data_ptr(), dv.data_ptr(), 3000, 0, 1.0,
                                  val.data_ptr(), st) == B.SC_ECSR
    out = val.cpu().numpy()
    assert np.isnan(out[17]) and np.all(np.isfinite(np.delete(out, 17)))


@pytest.mark.parametrize("symmetrize", [False, True])
@pytest.mark.parametrize("n,ne", [(50, 400), (3001, 40000), (7, 5), (100000, 300000)])
def test_coo_to_csr_matches_oracle(B, n, ne, symmetrize):
    rng = np.random.default_rng(n + ne)
    r, c = _edges(n, ne, 11)                     # random pairs: duplicates and self loops occur
    w = rng.uniform(0.1, 1.0, size=ne)
    rp, co, vo = B.sc_coo_to_csr(_dev(r, torch.int32), _dev(c, torch.int32), _dev(w, torch.float64), n, symmetrize)
    rp, co, vo = rp.cpu().numpy(), co.cpu().numpy(), vo.cpu().numpy()
    nself = int(np.sum(r == c))
    assert rp[0] == 0 and rp[-1] == (2 * ne - nself if symmetrize else ne) == co.size
    assert np.all(np.diff(rp) >= 0) and osim.csr_rows_sorted(rp, co)
    from scipy.sparse import csr_matrix, coo_matrix
    got = csr_matrix((vo, co, rp), shape=(n, n))
    if n <= 5000:
        np.testing.assert_allclose(got.toarray(), osim.coo_to_dense(r, c, w, n, symmetrize), rtol=1e-15, atol=0)
    else:   # same matrix through the library's own conversion (sums duplicates in an order of its own)
        rr, cc, ww = (np.concatenate([r, c[r != c]]), np.concatenate([c, r[r != c]]),
                      np.concatenate([w, w[r != c]])) if symmetrize else (r, c, w)
        ref = coo_matrix((ww, (rr, cc)), shape=(n, n)).tocsr()
        assert abs(got - ref).max() <= 1e-15
    # listed duplicates stay separate entries, in listing order
    if n == 7:
        for i in range(n):
            for j in np.unique(co[rp[i]:rp[i + 1]]):
                mine = vo[rp[i]:rp[i + 1]][co[rp[i]:rp[i + 1]] == j]
                listed = [w[e] for e in range(ne) if (r[e], c[e]) == (i, j)]
                if symmetrize:
                    listed += [w[e] for e in range(ne) if (c[e], r[e]) == (i, j) and r[e] != c[e]]
                assert sorted(mine.tolist()) == sorted(listed)


def _csr_by_sorting(r, c, w, n, symmetrize):
    """Rows sorted by column, equal entries in listing order (all listed entries before all mirrored ones)."""
    m = r != c
    if symmetrize:
        r, c, w = np.concatenate([r, c[m]]), np.concatenate([c, r[m]]), np.concatenate([w, w[m]])
    at = np.lexsort((np.arange(r.size), c, r))
    return np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]), c[at], w[at]


# buckets of one row and of many, a last bucket that is not full, rows at the limit of a bucket and beyond (radix sort),
# rows too long for the ranking, rows at the limit of the ranking, several of them in a bucket, more rows than there are
# buckets
@pytest.mark.parametrize("n,ne,hub", [(1, 3, 0), (1024, 260, 0), (1025, 5000, 0), (4099, 200_000, 4000), (4099, 200_000, 5000),
                                      (20_000, 20_000, 511), (20_000, 20_000, 513), (20_000, 20_000, 2049),
                                      (4, 700, 0), (7, 4000, 2000), (20_000, 520_000, 700), (20_000, 530_000, 700),
                                      (300, 90_000, 0), (70_001, 1_200_000, 0), (1_048_577, 3000, 0), (20_000_000, 3000, 0)])
@pytest.mark.parametrize("symmetrize", [False, True])
def test_coo_to_csr_over_its_ranges(B, n, ne, hub, symmetrize):
    rng = np.random.default_rng(n + ne + hub)
    r, c = _edges(n, ne, 5)
    if hub:
        r[:hub] = n // 2                      # one row with `hub` entries more
    w = rng.uniform(0.1, 1.0, size=ne)
    rp, co, vo = B.sc_coo_to_csr(_dev(r, torch.int32), _dev(c, torch.int32), _dev(w, torch.float64), n, symmetrize)
    rp0, co0, vo0 = _csr_by_sorting(r, c, w, n, symmetrize)
    np.testing.assert_array_equal(rp.cpu().numpy(), rp0)
    np.testing.assert_array_equal(co.cpu().numpy(), co0)
    np.testing.assert_array_equal(vo.cpu().numpy(), vo0)


# the bucketed pair kernel (data of 40 MB and more, eight pairs a row): against the oracle, with a ragged last bucket, odd
# dimensions and strides (scalar loads), an index out of range, one row in more pairs than a bucket holds, first rows by a
# power law (many buckets that are too small beside many that are empty), and both with indices out of range
@pytest.mark.parametrize("d,ldx,measure,twist", [(90, 90, 0, ""), (85, 85, 1, ""), (128, 129, 2, ""), (380, 380, 0, ""),
                                                 (90, 90, 0, "bad"), (100, 100, 1, "hub"), (90, 90, 2, "power"),
                                                 (101, 102, 0, "power bad"), (100, 100, 1, "hub bad"),
                                                 # two buckets a workgroup, every number of loads a row takes
                                                 (4, 4, 0, ""), (33, 33, 0, ""), (40, 40, 2, "hub"), (17, 17, 1, "power")])
def test_bucketed_edge_similarity_matches_oracle(B, d, ldx, measure, twist):
    n = 5_000_000 // d + 37
    rng = np.random.default_rng(d)
    big = rng.normal(size=(n, ldx)) + 1.5
    u, v = _edges(n, 8 * n + 11, 9)
    if "hub" in twist:
        u[::8] = 12
    if "power" in twist:
        u[:] = np.minimum((rng.random(u.size) ** 4 * n).astype(u.dtype), n - 1)
    if "bad" in twist:
        u[1234], v[99] = n, -1
    x = _dev(big, torch.float64)
    val = torch.zeros(u.size, dtype=torch.float64, device="cuda:0")
    st = torch.cuda.current_stream().cuda_stream
    du, dv = _dev(u, torch.int32), _dev(v, torch.int32)
    code = B.lib().sc_edge_similarity(x.data_ptr(), ldx, n, d, du.data_ptr(), dv.data_ptr(), u.size, measure, float(np.sqrt(d)),
                                      val.data_ptr(), st)
    got, ok = val.cpu().numpy(), np.ones(u.size, dtype=bool)
    assert code == (B.SC_ECSR if "bad" in twist else 0)
    if "bad" in twist:
        ok[[1234, 99]] = False
        assert np.isnan(got[~ok]).all()
    ref = osim.edge_similarity(big[:, :d], u[ok], v[ok], measure, float(np.sqrt(d)))
    # sums of d products: 2 d 2^-53 of the product of the norms, which is 1 in the value
    np.testing.assert_allclose(got[ok], ref, rtol=1e-12, atol=4.0 * d * 2.0 ** -53)


# where rows begin inside a line: every offset of the first row from a 16- and a 64-byte multiple, strides of every residue,
# rows of one chunk of loads and of several with every remainder, odd dimensions; pair by pair and in buckets
@pytest.mark.parametrize("d", [1, 2, 5, 7, 8, 9, 31, 32, 33, 40, 41, 63, 64, 66, 97, 130, 161])
@pytest.mark.parametrize("more,shift", [(0, 0), (1, 0), (2, 2), (3, 1), (0, 6), (4, 4)])
def test_edge_similarity_wherever_rows_begin(B, d, more, shift):
    n, ldx = 600, d + more
    rng = np.random.default_rng(d + 1000 * more)
    buf = torch.full((n * ldx + 64,), float("nan"), dtype=torch.float64, device="cuda:0")   # what is read beside the rows shows
    x = rng.normal(size=(n, d)) + 1.0
    rows = buf[shift:shift + n * ldx].view(n, ldx)
    rows[:, :d] = torch.from_numpy(x).cuda()
    u, v = _edges(n, 4001, 17)
    u[:4], v[:4] = [0, n - 1, 0, n - 1], [n - 1, 0, 0, n - 1]
    du, dv = _dev(u, torch.int32), _dev(v, torch.int32)
    val = torch.empty(u.size, dtype=torch.float64, device="cuda:0")
    for measure in (1, 2):
        assert B.lib().sc_edge_similarity(rows.data_ptr(), ldx, n, d, du.data_ptr(), dv.data_ptr(), u.size, measure,
                                          float(np.sqrt(d)), val.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
        ref = osim.edge_similarity(x, u, v, measure, float(np.sqrt(d)))
        np.testing.assert_allclose(val.cpu().numpy(), ref, rtol=1e-12, atol=4.0 * d * 2.0 ** -53)


@pytest.mark.parametrize("d,more,shift", [(90, 0, 2), (90, 1, 1), (61, 1, 6), (200, 0, 0), (5, 1, 2), (24, 8, 4)])
def test_bucketed_edge_similarity_wherever_rows_begin(B, d, more, shift):
    """The same values, to the last bit, as pair by pair: the sums are formed in one order."""
    n, ldx = 5_000_000 // d + 11, d + more
    gen = torch.Generator(device="cuda:0").manual_seed(d)
    buf = torch.full((n * ldx + 64,), float("nan"), dtype=torch.float64, device="cuda:0")
    rows = buf[shift:shift + n * ldx].view(n, ldx)
    rows[:, :d] = torch.randn((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    ne = 8 * n + 3
    u = torch.randint(0, n, (ne,), device="cuda:0", generator=gen, dtype=torch.int32)
    v = torch.where(torch.rand(ne, device="cuda:0", generator=gen) < 0.5, (u + 3) % n,
                    torch.randint(0, n, (ne,), device="cuda:0", generator=gen, dtype=torch.int32))

    def call(a, b, measure):
        val = torch.empty(a.numel(), dtype=torch.float64, device="cuda:0")
        assert B.lib().sc_edge_similarity(rows.data_ptr(), ldx, n, d, a.data_ptr(), b.data_ptr(), a.numel(), measure, 9.0,
                                          val.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
        return val

    for measure in (0, 2):
        bucketed = call(u, v, measure)
        few = ne // 4                                    # two pairs a row: pair by pair
        assert torch.equal(bucketed[:few], call(u[:few].contiguous(), v[:few].contiguous(), measure))


# entries listed several times side by side in a row, in every order; more rows than row and column have 32 bits for
@pytest.mark.parametrize("n,ne,cols", [(40, 8000, 40), (500, 30_000, 7), (5000, 200_000, 3000), (5_000_000, 700_000, 5_000_000)])
@pytest.mark.parametrize("symmetrize", [False, True])
def test_coo_to_csr_keeps_the_order_of_repeated_entries(B, n, ne, cols, symmetrize):
    rng = np.random.default_rng(n)
    r, c = rng.integers(0, n, size=ne), rng.integers(0, cols, size=ne)
    r[ne // 2:], c[ne // 2:] = r[:ne - ne // 2][::-1], c[:ne - ne // 2][::-1]
    w = np.arange(ne, dtype=np.float64)
    got = B.sc_coo_to_csr(_dev(r, torch.int32), _dev(c, torch.int32), _dev(w, torch.float64), n, symmetrize)
    for a, b in zip(got, _csr_by_sorting(r, c, w, n, symmetrize)):
        np.testing.assert_array_equal(a.cpu().numpy(), b)


def test_coo_to_csr_edge_cases(B):
    z32 = torch.empty(0, dtype=torch.int32, device="cuda:0")
    z64 = torch.empty(0, dtype=torch.float64, device="cuda:0")
    rp, co, vo = B.sc_coo_to_csr(z32, z32, z64, 5, True)
    assert rp.cpu().tolist() == [0] * 6 and co.numel() == 0
    with pytest.raises(B.ScError) as err:
        B.sc_coo_to_csr(_dev([0, 9], torch.int32), _dev([1, 2], torch.int32), _dev([1.0, 1.0], torch.float64), 5, True)
    assert err.value.code == B.SC_ECSR


def test_points_to_eigenpairs_chain(B):
    """Algorithm 1 -> Algorithm 2's conversion -> eigensolver, all on the device, from the pair list of the harness's
    kNN search: the CSR equals the harness's own graph and the eigenvalues the dense oracle's."""
    from oracle import dense
    cfg = wl.reduced(wl.CONFIGS[1], n=1500, components=5, k=5)
    pts, _ = wl.mixture_points(cfg)
    (rp, c, v, n), sigma = wl.knn_gaussian_graph(pts, cfg.k_nn, device="cpu")
    rows = np.repeat(np.arange(n), np.diff(rp))
    upper = rows < c                                 # every undirected edge once
    eu, ev = _dev(rows[upper], torch.int32), _dev(c[upper], torch.int32)
    w = B.sc_edge_similarity(_dev(pts, torch.float64), eu, ev, B.SC_SIM_EXP_DECAY, sigma)
    rp2, c2, v2 = B.sc_coo_to_csr(eu, ev, w, n, True)
    np.testing.assert_array_equal(rp2.cpu().numpy(), rp)
    np.testing.assert_array_equal(c2.cpu().numpy(), c)
    np.testing.assert_allclose(v2.cpu().numpy(), v, rtol=1e-12)
    evals, evecs, code, _ = B.sc_laplacian_eigsh(rp2, c2, v2, 5, 1e-10)
    lam_full, _ = dense.full_spectrum(rp, c, v)
    assert code == 0 and np.max(np.abs(evals.cpu().numpy() - lam_full[:5])) <= 1e-8


def test_a_full_block_cache_gives_way(B):
    """Blocks of 0.7 to 0.8 GB fill the cache (4 GiB); a later call's 0.5 GB block then takes the place of the oldest, so
    that more device memory is free after the call than before it (were it turned away, as much as before)."""
    B.sc_release_cache()
    gen = torch.Generator(device="cuda:0").manual_seed(1)

    def free_after_call(ne):                   # 24 bytes of scratch an entry, and the sort's
        r = torch.randint(0, 4000, (ne,), generator=gen, device="cuda:0", dtype=torch.int32)
        rp, co, vo = B.sc_coo_to_csr(r, r.flip(0).contiguous(), torch.ones(ne, dtype=torch.float64, device="cuda:0"), 4000,
                                     False)
        assert int(rp[-1]) == ne
        del r, co, vo
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]

    for ne in (30_000_000, 31_000_000, 32_000_000, 33_000_000, 34_000_000):
        before = free_after_call(ne)
    after = free_after_call(20_000_000)
    B.sc_release_cache()
    assert after - before > 100 << 20


def _all_but(nbytes, B):
    """Tensors that leave about `nbytes` of the device's memory free."""
    B.sc_release_cache()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    for _ in range(8):                      # what is reported as free comes down in steps
        more = torch.cuda.mem_get_info()[0] - nbytes
        if more < 8 << 20:
            break
        held.append(torch.empty(more, dtype=torch.uint8, device="cuda:0"))
    assert torch.cuda.mem_get_info()[0] <= nbytes + (8 << 20)
    return held


def test_edge_similarity_without_room_for_buckets(B):
    """235 MB of scratch for the buckets, 96 MB there: the values are formed pair by pair, the same as with buckets."""
    n, d, ne = 131_072, 48, 8_000_000
    gen = torch.Generator(device="cuda:0").manual_seed(4)
    x = torch.randn((n, d), dtype=torch.float64, device="cuda:0", generator=gen)
    u, v = (torch.randint(0, n, (ne,), device="cuda:0", generator=gen, dtype=torch.int32) for _ in range(2))
    ref = B.sc_edge_similarity(x, u, v, 0)
    got = torch.empty_like(ref)
    held = _all_but(96 << 20, B)
    code = B.lib().sc_edge_similarity(x.data_ptr(), d, n, d, u.data_ptr(), v.data_ptr(), ne, 0, 1.0, got.data_ptr(),
                                      torch.cuda.current_stream().cuda_stream)
    del held
    torch.cuda.empty_cache()
    assert code == B.SC_OK and torch.equal(got, ref)


def test_coo_to_csr_without_room_for_buckets(B):
    """184 MB of scratch for the buckets, 128 MB there: the sort does with less, and the result is the same."""
    n, ne = 16_000_000, 2_200_000
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    r, c = (torch.randint(0, n, (ne,), device="cuda:0", generator=gen, dtype=torch.int32) for _ in range(2))
    w = torch.rand(ne, dtype=torch.float64, device="cuda:0", generator=gen)
    ref = B.sc_coo_to_csr(r, c, w, n, False)
    got = [torch.empty_like(t) for t in ref]
    nnz = ctypes.c_int64(0)
    held = _all_but(128 << 20, B)
    code = B.lib().sc_coo_to_csr(r.data_ptr(), c.data_ptr(), w.data_ptr(), ne, n, 0, *(t.data_ptr() for t in got),
                                 ctypes.byref(nnz), torch.cuda.current_stream().cuda_stream)
    del held
    torch.cuda.empty_cache()
    assert code == B.SC_OK and nnz.value == ne and all(torch.equal(a, b) for a, b in zip(got, ref))


def test_calls_that_take_turns_keep_their_blocks(B):
    """Two calls of 2.5 and 2.2 GB of scratch do not fit the cache (4 GiB) together: the first one's block stays, so that
    neither call changes what is free, however often they take turns (were they to push one another out, the second would
    leave the difference)."""
    B.sc_release_cache()
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    rows = {ne: torch.randint(0, 4000, (ne,), generator=gen, device="cuda:0", dtype=torch.int32)
            for ne in (70_000_000, 60_000_000)}
    free = []
    for ne in (70_000_000, 60_000_000) * 5:
        r = rows[ne]
        out = B.sc_coo_to_csr(r, r, torch.ones(ne, dtype=torch.float64, device="cuda:0"), 4000, False)
        assert int(out[0][-1]) == ne
        del out
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        readings = []
        for _ in range(12):                 # what has just been given back is not always free at once
            readings.append(torch.cuda.mem_get_info()[0])
            time.sleep(0.05)
        free.append(max(readings))
    B.sc_release_cache()
    assert abs(np.median(free[0::2]) - np.median(free[1::2])) < 64 << 20, [f >> 20 for f in free]


def test_coo_to_csr_sorts_many_long_rows_every_time(B):
    """400 rows of 600 to 1,800 entries among short ones, thirty times: the slots come in another order each time, the result
    may not."""
    rng = np.random.default_rng(11)
    n = 20_000
    lens = rng.integers(600, 1800, size=400)
    r = np.concatenate([np.repeat(np.arange(400) * 50, lens), rng.integers(0, n, size=200_000)]).astype(np.int64)
    r = r[rng.permutation(r.size)]
    c = rng.integers(0, n, size=r.size)
    w = rng.uniform(0.1, 1.0, size=r.size)
    rp0, co0, vo0 = _csr_by_sorting(r, c, w, n, False)
    ref = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (rp0.astype(np.int64), co0.astype(np.int32), vo0)]
    dr, dc, dw = _dev(r, torch.int32), _dev(c, torch.int32), _dev(w, torch.float64)
    for _ in range(30):
        got = B.sc_coo_to_csr(dr, dc, dw, n, False)
        assert all(torch.equal(a, b) for a, b in zip(got, ref))
