"""GPU parity of the whole hot path (sc_laplacian_eigsh through the C ABI) against the CPU oracle.

Bars (eigenvalue / residual / angle) are in tests/parity.py.  Inside a multiple eigenvalue any
orthonormal basis is correct, so subspaces are compared per separated cluster; when k cuts a cluster the
GPU vectors must lie in the oracle's cluster space."""
import math
import os

import numpy as np
import pytest

from oracle import dense, lanczos, components, compare
from paper_1802_04450_amd import workloads as wl
from parity import check_against_oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1802_04450_amd import binding
    binding.lib()
    return binding


def solve(B, graph, k, tol, **kw):
    rp, c, v, n = graph
    drp, dc, dv = B.csr_to_device(rp, c, v)
    evals, evecs, code, stats = B.sc_laplacian_eigsh(drp, dc, dv, k, tol, **kw)
    return evals.cpu().numpy(), evecs.cpu().numpy().T.copy(), code, stats


CLOSED_FORM = [
    ("ring50", lambda: wl.ring(50), 5),
    ("path60", lambda: wl.path(60), 5),
    ("hypercube6", lambda: wl.hypercube(6), 7),
    ("complete12", lambda: wl.complete(12), 4),
    ("bipartite4x7", lambda: wl.complete_bipartite(4, 7), 3),
    ("union", lambda: wl.disjoint_union(wl.ring(9), wl.ring(14), wl.path(11), wl.random_weighted_connected(40, 80, 7),
                                        wl.complete(6)), 7),
    ("ring301", lambda: wl.ring(301), 9),
]


@pytest.mark.parametrize("name,make,k", CLOSED_FORM, ids=[c[0] for c in CLOSED_FORM])
def test_closed_form_graphs_match_dense_oracle(B, name, make, k):
    g = make()
    rp, c, v, n = g
    lam_full, vec_full = dense.full_spectrum(rp, c, v)
    lam, vec, code, stats = solve(B, g, k, 1e-10)
    assert code == B.SC_OK, stats
    check_against_oracle(g, k, lam, vec, lam_full[:k + 1], vec_full[:, :k])


@pytest.mark.parametrize("block", [1, 2, 4, 8, 16, 32])
def test_block_sizes_on_multiplicity_graph(B, block):
    # 6 components -> 6 zeros; then the rings' double eigenvalues
    g = wl.disjoint_union(*[wl.ring(20 + 3 * t) for t in range(6)])
    rp, c, v, n = g
    lam_full, vec_full = dense.full_spectrum(rp, c, v)
    k = 9
    lam, vec, code, stats = solve(B, g, k, 1e-10, block=block, m=max(60, k + 3 * block))
    assert code == B.SC_OK and stats["block"] == block
    check_against_oracle(g, k, lam, vec, lam_full[:k + 1], vec_full[:, :k])
    assert np.sum(np.abs(lam) < 1e-9) == 6


def test_config1_full_size(B):
    cfg = wl.CONFIGS[1]
    g, label, _ = wl.build_config_graph(cfg, device="cpu")
    rp, c, v, n = g
    lam_full, vec_full = dense.full_spectrum(rp, c, v)
    lam, vec, code, stats = solve(B, g, cfg.k, cfg.tol)
    assert code == B.SC_OK, stats
    out = check_against_oracle(g, cfg.k, lam, vec, lam_full[:cfg.k + 1], vec_full[:, :cfg.k],
                               cluster_basis=components.null_space(rp, c, v))
    assert np.max(np.abs(lam)) < 1e-9
    # also against the Lanczos oracle, and for more pairs than components (k = 12 > 8)
    lam_o, vec_o = lanczos.lanczos_smallest(rp, c, v, k=13, tol=1e-11, seed=3)
    lam2, vec2, code2, _ = solve(B, g, 12, cfg.tol)
    assert code2 == B.SC_OK
    check_against_oracle(g, 12, lam2, vec2, lam_o, vec_o)


def test_seed_independence_and_determinism(B):
    cfg = wl.reduced(wl.CONFIGS[1], n=1500, components=6, k=8)
    g, _, _ = wl.build_config_graph(cfg, device="cpu")
    rp, c, v, n = g
    lam_full, vec_full = dense.full_spectrum(rp, c, v)
    a = solve(B, g, 8, 1e-10, seed=1)
    b = solve(B, g, 8, 1e-10, seed=1)
    c2 = solve(B, g, 8, 1e-10, seed=2)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])      # bitwise reproducible
    for out in (a, c2):
        check_against_oracle(g, 8, out[0], out[1], lam_full[:9], vec_full[:, :8])


REDUCED = [
    # (config id, n, components, k, m)   -- reduced instances of the large workloads, same recipe
    (2, 6000, 12, 12, 48),
    (3, 8000, 20, 10, 40),      # k < number of components: k cuts the null cluster
    (5, 6000, 30, 30, 96),
]


@pytest.mark.parametrize("cid,n,comps,k,m", REDUCED, ids=[f"cfg{r[0]}_n{r[1]}" for r in REDUCED])
def test_reduced_workloads_against_lanczos_and_component_oracles(B, cid, n, comps, k, m):
    cfg = wl.reduced(wl.CONFIGS[cid], n=n, components=comps, k=k, m=m)
    g, label, _ = wl.build_config_graph(cfg, device="cuda")
    rp, c, v, nn = g
    ncomp, _ = components.component_labels(rp, c, v)
    lam_o, vec_o = lanczos.lanczos_smallest(rp, c, v, k=k + 1, tol=1e-10, m=max(m, 2 * (k + 1)), seed=11)
    lam, vec, code, stats = solve(B, g, k, cfg.tol, m=m)
    assert code == B.SC_OK, stats
    basis = components.null_space(rp, c, v) if k <= ncomp else None
    check_against_oracle(g, k, lam, vec, lam_o, vec_o, cluster_basis=basis)
    assert np.sum(np.abs(lam) < 1e-8) == min(k, ncomp)


def test_block32_on_reduced_large_k_workload(B):
    """The block size the library picks for the reorthogonalization-dominated workload (n >= 300,000 and k >= 1000:
    32 columns per step), end to end on a reduced instance of the same recipe, against the Lanczos oracle and the
    closed-form null space."""
    cfg = wl.reduced(wl.CONFIGS[5], n=12000, components=48, k=48, m=160)
    g, label, _ = wl.build_config_graph(cfg, device="cuda")
    rp, c, v, nn = g
    ncomp, _ = components.component_labels(rp, c, v)
    k = cfg.k
    lam_o, vec_o = lanczos.lanczos_smallest(rp, c, v, k=k + 1, tol=1e-10, m=max(cfg.m, 2 * (k + 1)), seed=11)
    lam, vec, code, stats = solve(B, g, k, cfg.tol, m=cfg.m, block=32)
    assert code == B.SC_OK and stats["block"] == 32, stats
    basis = components.null_space(rp, c, v) if k <= ncomp else None
    check_against_oracle(g, k, lam, vec, lam_o, vec_o, cluster_basis=basis)
    assert np.sum(np.abs(lam) < 1e-8) == min(k, ncomp)


def test_reduced_blob_workload_3d(B):
    """Config-4 recipe at reduced size: anisotropic 3-D blobs, near-null ladder above the zeros."""
    cfg = wl.reduced(wl.CONFIGS[4], n=20000, components=6, k=6, m=60)
    g, label, _ = wl.build_config_graph(cfg, device="cuda")
    rp, c, v, nn = g
    ncomp, _ = components.component_labels(rp, c, v)
    k = 6
    lam, vec, code, stats = solve(B, g, k, cfg.tol, m=cfg.m)
    assert code == B.SC_OK, stats
    lam_c, vec_c = components.smallest_eigenpairs(rp, c, v, k + 1, dense_limit=1500, tol=1e-10)
    check_against_oracle(g, k, lam, vec, lam_c, vec_c)


def test_maxiter_gives_not_converged_with_finite_output(B):
    g = wl.random_weighted_connected(3000, 9000, seed=9)
    lam, vec, code, stats = solve(B, g, 6, 1e-13, m=24, block=2, maxiter=1)
    assert code == B.SC_NOT_CONVERGED
    assert np.all(np.isfinite(lam)) and np.all(np.diff(lam) >= 0)
    assert compare.orthonormality_defect(vec) < 1e-9


def test_solver_rejects_bad_inputs_on_device(B):
    rp = np.array([0, 1, 1, 2, 3], dtype=np.int64)
    c = np.array([2, 0, 2], dtype=np.int32)
    v = np.array([1.0, 1.0, 1.0])
    drp, dc, dv = B.csr_to_device(rp, c, v)
    with pytest.raises(B.ScError) as e:
        B.sc_laplacian_eigsh(drp, dc, dv, 1, 1e-8, m=4, block=1)
    assert e.value.code == B.SC_EZERODEG
    bad = torch.tensor([2, 0, 9], dtype=torch.int32, device="cuda")
    with pytest.raises(B.ScError) as e:
        B.sc_laplacian_eigsh(drp, bad, dv, 1, 1e-8, m=4, block=1)
    assert e.value.code == B.SC_ECSR


def test_config2_full_size_bench_configuration(B):
    """The benchmark workload at full size (n = 100,000, k = 100, m = 200, tol 1e-8) in the launch
    configuration bench.py times.  Reference: the closed-form null space of the 100 components (exact),
    eigenvalue 0 with multiplicity 100; residuals recomputed on the host."""
    cfg = wl.CONFIGS[2]
    g, label, _ = wl.build_config_graph(cfg, device="cuda")
    rp, c, v, n = g
    ncomp, _ = components.component_labels(rp, c, v)
    assert ncomp == cfg.components
    lam, vec, code, stats = solve(B, g, cfg.k, cfg.tol, m=cfg.m)
    assert code == B.SC_OK, stats
    basis = components.null_space(rp, c, v)
    out = check_against_oracle(g, cfg.k, lam, vec, np.zeros(cfg.k), basis, cluster_basis=basis)
    assert np.max(compare.principal_angles(vec, basis)) <= 1e-5
    print("config2", stats, out)


def _interleaved_components_graph():
    parts = [wl.ring(30), wl.path(41), wl.random_weighted_connected(200, 500, 3), wl.hypercube(5), wl.complete(9),
             wl.random_weighted_connected(333, 900, 4)]
    g = wl.disjoint_union(*parts)
    perm = np.random.default_rng(12).permutation(g[3])
    return wl.relabel(g, perm), len(parts)


def test_internal_reordering_is_invisible(B):
    """The component pass renumbers nodes internally; outputs must be in the caller's numbering and agree with
    the run that uses the CSR as given."""
    g, ncomp = _interleaved_components_graph()
    rp, c, v, n = g
    lam_full, vec_full = dense.full_spectrum(rp, c, v)
    k = 9
    a = solve(B, g, k, 1e-10)
    b = solve(B, g, k, 1e-10, flags=B.SC_FLAG_NO_REORDER)
    assert a[3]["components"] == ncomp == components.component_labels(rp, c, v)[0]
    assert b[3]["components"] == 0
    for out in (a, b):
        assert out[2] == B.SC_OK
        check_against_oracle(g, k, out[0], out[1], lam_full[:k + 1], vec_full[:, :k])


def test_zero_weight_entries_do_not_connect(B):
    # two rings joined by one explicit zero-weight edge: still two components, two zero eigenvalues
    g = wl.disjoint_union(wl.ring(40), wl.ring(50))
    rp, c, v, n = g
    extra_u, extra_v = np.array([3]), np.array([60])
    rows = np.repeat(np.arange(n), np.diff(rp))
    g2 = wl.coo_to_csr(np.concatenate([rows, extra_u, extra_v]), np.concatenate([c.astype(np.int64), extra_v, extra_u]),
                       np.concatenate([v, [0.0, 0.0]]), n, sum_duplicates=False)
    lam, vec, code, stats = solve(B, g2, 3, 1e-10)
    assert code == B.SC_OK and stats["components"] == 2 == components.component_labels(*g2[:3])[0]
    lam_full, vec_full = dense.full_spectrum(*g2[:3])
    check_against_oracle(g2, 3, lam, vec, lam_full[:4], vec_full[:, :3])


@pytest.mark.parametrize("k", [4, 6, 9])
def test_component_nullspace_option(B, k):
    """Optional pre-pass: the closed-form null vectors of the components are locked first (k below, equal to
    and above the number of components)."""
    g, ncomp = _interleaved_components_graph()
    rp, c, v, n = g
    lam_full, vec_full = dense.full_spectrum(rp, c, v)
    lam, vec, code, stats = solve(B, g, k, 1e-10, flags=B.SC_FLAG_COMPONENT_NULLSPACE)
    assert code == B.SC_OK
    basis = components.null_space(rp, c, v) if k <= ncomp else None
    if k == ncomp:
        check_against_oracle(g, k, lam, vec, lam_full[:k + 1], vec_full[:, :k], cluster_basis=basis)
    else:
        check_against_oracle(g, k, lam, vec, lam_full[:k] if k < ncomp else lam_full[:k + 1],
                             vec_full[:, :k], cluster_basis=basis)
    assert np.sum(np.abs(lam) < 1e-12) == min(k, ncomp)


@pytest.mark.parametrize("flags", ["NO_START_FILTER", "FINAL_RR", "NO_START_FILTER|FINAL_RR"])
def test_option_flags_give_the_same_answer(B, flags):
    """The start-block filter and the final Rayleigh-Ritz step are accelerations/refinements: with either switched
    the other way the answer must meet the same bars (multiplicity graph and a reduced clustered workload)."""
    f = 0
    for name in flags.split("|"):
        f |= getattr(B, "SC_FLAG_" + name)
    g = wl.disjoint_union(*[wl.ring(20 + 3 * t) for t in range(6)])
    lam_full, vec_full = dense.full_spectrum(*g[:3])
    lam, vec, code, stats = solve(B, g, 9, 1e-10, m=60, flags=f)
    assert code == B.SC_OK
    if f & B.SC_FLAG_NO_START_FILTER:
        assert stats["filter_steps"] == 0
    check_against_oracle(g, 9, lam, vec, lam_full[:10], vec_full[:, :9])
    cfg = wl.reduced(wl.CONFIGS[2], n=6000, components=12)
    g, label, sigma = wl.build_config_graph(cfg, device="cuda")
    k = 12
    lam, vec, code, stats = solve(B, g, k, 1e-8, flags=f)
    assert code == B.SC_OK
    ncomp, _ = components.component_labels(*g[:3])
    assert ncomp >= k              # the reduced workload keeps its clusters disconnected: k exact zeros
    basis = components.null_space(*g[:3])
    assert np.max(np.abs(lam)) <= 1e-8
    assert np.max(compare.residual_norms(*g[:3], lam, vec)) <= 1e-6
    assert np.max(compare.containment_defect(vec, basis)) <= 1e-5
    assert compare.orthonormality_defect(vec) <= 1e-9


def test_start_filter_is_used_on_clustered_workload(B):
    """On a union of components (eigenvalue 0 with multiplicity > block size) the re-injection blocks are filtered and
    the phases after the first need only a few Lanczos steps."""
    cfg = wl.reduced(wl.CONFIGS[2], n=6000, components=24)
    g, label, sigma = wl.build_config_graph(cfg, device="cuda")
    lam, vec, code, with_filter = solve(B, g, 24, 1e-8, block=4)
    assert code == B.SC_OK and with_filter["filter_steps"] > 0
    lam2, vec2, code2, without = solve(B, g, 24, 1e-8, block=4, flags=B.SC_FLAG_NO_START_FILTER)
    assert code2 == B.SC_OK and without["filter_steps"] == 0
    assert with_filter["block_steps"] < without["block_steps"]
    assert np.max(np.abs(lam)) <= 1e-8 and np.max(np.abs(lam2)) <= 1e-8


def test_block_products_through_the_resident_form(B, monkeypatch):
    """Where every diagonal block of the renumbered operator has work items of the LDS-resident filter, the single
    products of the block steps run as a one-step recurrence of that form.  Both ways of multiplying must pass the
    parity bars against the component oracle and agree with each other to the tolerance."""
    cfg = wl.reduced(wl.CONFIGS[5], n=16000, components=64)
    g, label, sigma = wl.build_config_graph(cfg, device="cuda")
    rp, c, v, n = g
    basis = components.null_space(rp, c, v)
    k = basis.shape[1]
    assert 64 <= k <= 80
    monkeypatch.setenv("SCEIG_FORCE_RESIDENT", "1")   # small graph: the cost model would leave the form out
    results = []
    for off in (False, True):
        if off:
            monkeypatch.setenv("SCEIG_NO_RESIDENT_PRODUCT", "1")
        before = B.sc_counter(B.SC_COUNTER_RESIDENT_FILTERS)
        lam, vec, code, stats = solve(B, g, k, 1e-9, block=16)
        assert code == B.SC_OK and stats["block_steps"] > 0, stats
        assert B.sc_counter(B.SC_COUNTER_RESIDENT_FILTERS) > before       # the resident plan was in use
        assert np.max(np.abs(lam)) <= 1e-9
        assert compare.residual_norms(rp, c, v, lam, vec).max() <= 1e-8
        assert np.max(compare.containment_defect(vec, basis)) <= 1e-7
        assert compare.orthonormality_defect(vec) <= 1e-10
        results.append(lam)
    assert np.max(np.abs(results[0] - results[1])) <= 1e-9


def test_single_precision_filter_steps_change_nothing_that_is_returned(B, monkeypatch):
    """The one-launch start-block filter runs all steps but a double-precision tail in single precision.  The filter only
    prepares a start block, so the returned pairs must meet the same bars with and without it, and the phases must
    not need more block steps than a couple (the later steps damp what the rounding of the earlier ones adds)."""
    cfg = wl.reduced(wl.CONFIGS[5], n=16000, components=64)
    g, label, sigma = wl.build_config_graph(cfg, device="cuda")
    rp, c, v, n = g
    basis = components.null_space(rp, c, v)
    k = basis.shape[1]
    monkeypatch.setenv("SCEIG_FORCE_RESIDENT", "1")   # small graph: the cost model would leave the form out
    runs = []
    for tail in (None, "1000"):
        if tail:
            monkeypatch.setenv("SCEIG_FILTER_FP64_TAIL", tail)   # every step in double precision
        lam, vec, code, stats = solve(B, g, k, 1e-9, block=32, m=k + 128)
        assert code == B.SC_OK and stats["filter_steps"] > 0, stats
        assert np.max(np.abs(lam)) <= 1e-9
        assert compare.residual_norms(rp, c, v, lam, vec).max() <= 1e-8
        assert np.max(compare.containment_defect(vec, basis)) <= 1e-7
        assert compare.orthonormality_defect(vec) <= 1e-10
        runs.append(stats)
    assert runs[0]["block_steps"] <= runs[1]["block_steps"] + 2, (runs[0], runs[1])


def test_filter_interval_with_a_wrong_spectrum_bottom(B, monkeypatch):
    """The start-block filters damp [estimate of the spectrum's bottom, a] instead of [-1, a].  Isolated eigenvalues at
    the bottom (the -1 of a bipartite component, here K_{3,4}: 7 of 12,007 nodes) are found by the first unfiltered
    steps; what those steps underestimate is the edge of a bulk, by a bounded amount that the margin covers.  This
    test makes the estimate wrong on purpose (-0.05 and +0.2 where the spectrum ends at -0.3 and -1): the filters then
    amplify what lies below it, the solver sees Ritz values below its estimate and lowers it, and all k null vectors
    still come back within the parity bars - a wrong estimate costs block steps, never correctness."""
    cfg = wl.reduced(wl.CONFIGS[2], n=12000, components=40)
    g, label, sigma = wl.build_config_graph(cfg, device="cuda")
    g = wl.disjoint_union(g, wl.complete_bipartite(3, 4))
    rp, c, v, n = g
    ncomp, _ = components.component_labels(rp, c, v)
    assert ncomp == 41
    basis = components.null_space(rp, c, v)
    lam0, vec0, code0, stats0 = solve(B, g, 41, 1e-8, block=16)
    assert code0 == B.SC_OK
    for forced in ("-0.05", "0.2"):
        monkeypatch.setenv("SCEIG_SPECTRUM_BOTTOM", forced)
        lam, vec, code, stats = solve(B, g, 41, 1e-8, block=16)
        assert code == B.SC_OK and stats["filter_steps"] > 0, stats
        assert np.max(np.abs(lam)) <= 1e-8
        assert compare.residual_norms(rp, c, v, lam, vec).max() <= 1e-7
        assert np.max(compare.containment_defect(vec, basis)) <= 1e-6
        assert compare.orthonormality_defect(vec) <= 1e-10


# the one-launch filter with 32 and 16 columns, the products of a block twice as wide with 16 and 8; blocks of 4 make no pairs
@pytest.mark.parametrize("config,n,comps,block,tol,resident", [(2, 40_000, 200, 32, 1e-8, True), (2, 60_001, 300, 32, 1e-7, True),
                                                               (5, 100_000, 400, 16, 1e-7, True), (2, 20_000, 120, 16, 1e-8, False),
                                                               (2, 12_003, 60, 8, 1e-7, False), (2, 30_000, 20, 4, 1e-8, False)])
def test_two_start_blocks_at_once(B, monkeypatch, config, n, comps, block, tol, resident):
    """Start blocks made in pairs: as many phases as one by one, and the null space as well resolved."""
    cfg = wl.reduced(wl.CONFIGS[config], n=n, components=comps)
    g, label, sigma = wl.build_config_graph(cfg, device="cuda")
    rp, c, v, n = g
    assert components.component_labels(rp, c, v)[0] == comps
    basis = components.null_space(rp, c, v)
    monkeypatch.setenv("SCEIG_PAIR_MIN_WORK", "1")
    runs = []
    for alone in ("", "1"):
        if alone:
            monkeypatch.setenv("SCEIG_NO_START_PAIRS", alone)
        before = [B.sc_counter(x) for x in (B.SC_COUNTER_START_PAIRS, B.SC_COUNTER_RESIDENT_FILTERS)]
        lam, vec, code, stats = solve(B, g, comps, tol, block=block, m=comps + 8 * block + 40)
        after = [B.sc_counter(x) for x in (B.SC_COUNTER_START_PAIRS, B.SC_COUNTER_RESIDENT_FILTERS)]
        assert code == B.SC_OK, stats
        assert (after[0] > before[0]) == (not alone and block >= 8), stats
        assert (after[1] > before[1]) == resident, stats
        assert np.max(np.abs(lam)) <= tol
        assert compare.residual_norms(rp, c, v, lam, vec).max() <= 10 * tol
        assert np.max(compare.containment_defect(vec, basis)) <= 100 * tol
        assert compare.orthonormality_defect(vec) <= 1e-10
        runs.append(stats)
    assert runs[0]["phases"] <= runs[1]["phases"] + 1, runs


def test_release_cache_between_calls(B):
    """Workspace blocks are kept between calls; giving them back must not change any later result."""
    g = wl.disjoint_union(*[wl.ring(20 + 3 * t) for t in range(6)])
    lam1, vec1, code1, _ = solve(B, g, 9, 1e-10, m=60, seed=5)
    lam2, vec2, code2, _ = solve(B, g, 9, 1e-10, m=60, seed=5)        # served from the kept blocks
    assert B.sc_release_cache() == B.SC_OK
    lam3, vec3, code3, _ = solve(B, g, 9, 1e-10, m=60, seed=5)        # fresh allocations again
    assert code1 == code2 == code3 == B.SC_OK
    assert np.array_equal(lam1, lam2) and np.array_equal(lam1, lam3)
    assert np.array_equal(vec1, vec2) and np.array_equal(vec1, vec3)


@pytest.mark.parametrize("extra", [0, "FINAL_RR"])
def test_random_walk_vectors_of_the_papers_laplacian(B, extra):
    """SC_FLAG_RANDOM_WALK_VECTORS: eigenvectors of L_n = D^-1 L (Section II Steps 2-3).  Checked against the
    definition (L_n u = lambda u entry by entry), D-orthonormality, constancy on components for lambda = 0, and
    against the symmetric-form output of the same solve scaled by the oracle."""
    from oracle import laplacian
    parts = [wl.ring(9), wl.path(14), wl.random_weighted_connected(30, 60, 5), wl.complete(5), wl.ring(21)]
    g = wl.disjoint_union(*parts)
    g = wl.relabel(g, np.random.default_rng(8).permutation(g[3]))
    rp, c, v, n = g
    k = 8
    f = B.SC_FLAG_RANDOM_WALK_VECTORS | (getattr(B, "SC_FLAG_" + extra) if extra else 0)
    lam, u, code, _ = solve(B, g, k, 1e-10, flags=f, seed=3)
    lam_v, vec, code_v, _ = solve(B, g, k, 1e-10, flags=f & ~B.SC_FLAG_RANDOM_WALK_VECTORS, seed=3)
    assert code == code_v == B.SC_OK
    assert np.array_equal(lam, lam_v)
    assert np.max(np.abs(u - laplacian.random_walk_vectors(rp, c, v, vec))) <= 1e-14      # one scaling by s = d^-1/2
    lam_full, _ = dense.full_spectrum(rp, c, v)
    assert np.max(np.abs(lam - lam_full[:k])) <= 1e-8
    assert np.max(np.abs(laplacian.apply_random_walk_laplacian(rp, c, v, u) - u * lam[None, :])) <= 1e-6
    d = laplacian.degrees(rp, c, v)
    assert np.max(np.abs(u.T @ (d[:, None] * u) - np.eye(k))) <= 1e-9
    ncomp, label = components.component_labels(rp, c, v)
    for t in range(ncomp):
        for comp in range(ncomp):
            assert np.ptp(u[label == comp, t]) <= 1e-8


def _random_family(seed):
    """Seeded small graphs that exercise the solver's decisions: connected graphs without a gap, unions of
    components of uneven size (multiplicity above, at and below the block size), k below / at / above the
    multiplicity, tight and generous basis budgets."""
    rng = np.random.default_rng(1000 + seed)
    kind = seed % 4
    if kind == 0:                                   # one connected graph, dense spectrum
        n = int(rng.integers(80, 400))
        g = wl.random_weighted_connected(n, int(rng.integers(2, 6)) * n, seed)
        k = int(rng.integers(2, 12))
    elif kind == 1:                                 # many small components, k cuts the null cluster
        parts = [wl.random_weighted_connected(int(rng.integers(6, 40)), 60, seed * 31 + t) for t in range(int(rng.integers(5, 30)))]
        g = wl.disjoint_union(*parts)
        k = int(rng.integers(2, len(parts)))
    elif kind == 2:                                 # k beyond the number of components
        parts = [wl.ring(int(rng.integers(8, 30))) if t % 2 else wl.random_weighted_connected(int(rng.integers(10, 50)), 90, seed * 17 + t)
                 for t in range(int(rng.integers(3, 12)))]
        g = wl.disjoint_union(*parts)
        k = len(parts) + int(rng.integers(1, 6))
    else:                                           # k equal to the multiplicity, strongly uneven sizes
        sizes = [int(s) for s in rng.integers(5, 120, size=int(rng.integers(4, 20)))]
        parts = [wl.random_weighted_connected(s, 3 * s, seed * 13 + t) for t, s in enumerate(sizes)]
        g = wl.disjoint_union(*parts)
        k = len(parts)
    g = wl.relabel(g, rng.permutation(g[3]))
    n = g[3]
    k = max(1, min(k, n - 2))
    m = int(min(n, k + rng.choice([8, 24, 60]) + 3))
    return g, k, m


@pytest.mark.parametrize("seed", range(int(os.environ.get("SCEIG_RANDOM_CASES", "24"))))
def test_random_graph_families_against_dense_oracle(B, seed):
    g, k, m = _random_family(seed)
    rp, c, v, n = g
    lam_full, vec_full = dense.full_spectrum(rp, c, v)
    try:
        lam, vec, code, stats = solve(B, g, k, 1e-10, m=m, seed=seed)
    except B.ScError as e:                          # the budget can be too tight for any block size: a domain error
        assert e.args[0] == B.SC_EDOMAIN and k + 3 > m
        return
    assert code == B.SC_OK, stats
    check_against_oracle(g, k, lam, vec, lam_full[:k + 1], vec_full[:, :k])


def test_row_normalized_embedding(B):
    """SC_FLAG_ROW_NORMALIZE: the rows of the output (the points k-means clusters, Section II Step 4) have unit norm and
    equal the rows of the plain output divided by their norm; on a union of components with k = their number the rows
    of one component coincide and rows of different components are orthogonal."""
    parts = [wl.ring(9), wl.path(14), wl.random_weighted_connected(30, 60, 5), wl.complete(5), wl.ring(21)]
    g = wl.disjoint_union(*parts)
    g = wl.relabel(g, np.random.default_rng(9).permutation(g[3]))
    rp, c, v, n = g
    k = len(parts)
    _, vec, code, _ = solve(B, g, k, 1e-10, seed=3)
    for f in (B.SC_FLAG_ROW_NORMALIZE, B.SC_FLAG_ROW_NORMALIZE | B.SC_FLAG_RANDOM_WALK_VECTORS):
        _, emb, code2, _ = solve(B, g, k, 1e-10, seed=3, flags=f)
        assert code == code2 == B.SC_OK
        assert np.max(np.abs(np.linalg.norm(emb, axis=1) - 1.0)) <= 1e-14
        assert np.max(np.abs(emb - vec / np.linalg.norm(vec, axis=1, keepdims=True))) <= 1e-13
        _, label = components.component_labels(rp, c, v)
        gram = emb @ emb.T
        same = label[:, None] == label[None, :]
        assert np.max(np.abs(gram[same] - 1.0)) <= 1e-7 and np.max(np.abs(gram[~same])) <= 1e-7


def test_workspace_estimate_covers_what_a_solve_allocates(B):
    """sc_workspace_bytes against the device memory that actually leaves the free pool during a solve (the library
    keeps its blocks cached afterwards, so the drop in free memory is what the solve took)."""
    cfg = wl.reduced(wl.CONFIGS[2], n=60000, components=60, k=60)
    g, _, _ = wl.build_config_graph(cfg, device="cuda")
    rp, c, v, n = g
    drp, dc, dv = B.csr_to_device(rp, c, v)
    B.sc_release_cache()
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    evals, evecs, code, stats = B.sc_laplacian_eigsh(drp, dc, dv, cfg.k, 1e-8, m=cfg.m)
    torch.cuda.synchronize()
    free1, _ = torch.cuda.mem_get_info()
    taken = free0 - free1 - evals.numel() * 8 - evecs.numel() * 8      # the outputs are torch's, allocated in between
    est = B.sc_workspace_bytes(n, int(rp[-1]), cfg.k, m=cfg.m)
    assert code == B.SC_OK
    assert 0.8 * taken <= est <= 1.5 * taken + (32 << 20), (taken, est)
    B.sc_release_cache()


@pytest.mark.parametrize("k,block,no_filter,most", [(10, 8, False, 30), (10, 8, True, 60), (10, 2, False, None),
                                                    (7, 8, False, None), (1, 1, False, None), (12, 4, False, None)])
def test_check_phase(B, k, block, no_filter, most):
    """The check phase answers whether something larger is left: where the wanted values stand clear of the rest it does so
    in a few steps (the locking phases take the others; 80 and more until the rest's largest pair converges), where k cuts
    close values it goes on, and the answer is the oracle's either way."""
    g, _ = wl.stochastic_block_model(1200, 10, 0.33, 0.002, 3)
    rp, c, v, n = g
    lam0, vec0 = dense.smallest_eigenpairs(rp, c, v, k + 1)
    lam, vec, code, stats = solve(B, g, k, 1e-10, block=block, m=120 if no_filter else 80,
                                  flags=B.SC_FLAG_NO_START_FILTER if no_filter else 0)
    assert code == B.SC_OK
    check_against_oracle(g, k, lam, vec, lam0, vec0)
    assert most is None or stats["block_steps"] <= most, stats


# k = 10: what is missing stands clear of the rest (the largest, one in the middle, the last); k = 7 and 14: among close values
@pytest.mark.parametrize("k,block,missing,no_filter", [(10, 1, 0, False), (10, 2, 4, False), (10, 8, 0, False), (10, 8, 9, False),
                                                       (10, 16, 4, False), (10, 16, 9, False), (10, 8, 9, True),
                                                       (10, 2, 9, True), (10, 16, 0, True), (7, 8, 6, False), (7, 2, 6, True),
                                                       (14, 16, 13, False), (14, 1, 12, False)])
def test_check_phase_finds_what_the_locked_pairs_lack(B, k, block, missing, no_filter, monkeypatch):
    """One of the k largest is given up for the one after them before the check phase, which has to bring it back."""
    g, _ = wl.stochastic_block_model(1200, 10, 0.33, 0.002, 3)
    rp, c, v, n = g
    lam0, vec0 = dense.smallest_eigenpairs(rp, c, v, k + 1)
    flags = B.SC_FLAG_NO_START_FILTER if no_filter else 0
    monkeypatch.setenv("SCEIG_UNLOCK", str(missing))
    wrong, _, code, _ = solve(B, g, k, 1e-10, block=block, m=128, flags=flags | B.SC_FLAG_NO_VERIFY)
    assert code == B.SC_OK
    assert np.max(np.abs(wrong - np.delete(lam0, missing))) <= 1e-9      # it is missing
    lam, vec, code, _ = solve(B, g, k, 1e-10, block=block, m=128, flags=flags)
    assert code == B.SC_OK
    check_against_oracle(g, k, lam, vec, lam0, vec0)


def test_setup_that_runs_out_of_memory_after_the_degrees(B):
    """The setup of a wide solve asks for its scaled values while the marks of the degree pass are on their way to the host:
    without room for them the call is refused, and the next one is not disturbed by it."""
    n, half = 200_000, 150
    step = torch.cat([torch.arange(-half, 0, device="cuda:0"), torch.arange(1, half + 1, device="cuda:0")])
    col = (torch.arange(n, device="cuda:0")[:, None] + step[None, :]) % n
    col = col.sort(dim=1).values.reshape(-1).to(torch.int32)
    nnz = col.numel()
    rowptr = torch.arange(n + 1, dtype=torch.int64, device="cuda:0") * (2 * half)
    val = torch.ones(nnz, dtype=torch.float64, device="cuda:0")
    B.sc_release_cache()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    # the renumbering takes 12 bytes an entry and about 60 a row, the scaled values 8 an entry
    room = 12 * nnz + 60 * n + (200 << 20)
    assert room < 20 * nnz
    held = []
    for _ in range(8):                          # what is reported as free comes down in steps
        more = torch.cuda.mem_get_info()[0] - room
        if more < 8 << 20:
            break
        held.append(torch.empty(more, dtype=torch.uint8, device="cuda:0"))
    with pytest.raises(B.ScError) as e:
        B.sc_laplacian_eigsh(rowptr, col, val, 16, 1e-6, block=16)
    del held
    B.sc_release_cache()
    torch.cuda.empty_cache()
    assert e.value.code == B.SC_ENOMEM
    g = wl.disjoint_union(wl.ring(150), wl.random_weighted_connected(400, 900, 2))
    lam0, vec0 = dense.smallest_eigenpairs(*g[:3], 9)
    lam, vec, code, _ = solve(B, g, 8, 1e-10, block=16)
    assert code == B.SC_OK
    check_against_oracle(g, 8, lam, vec, lam0, vec0)


@pytest.mark.parametrize("block", [2, 8, 16])
def test_check_phase_with_weights_below_zero(B, block):
    """A few weights below zero move the spectrum of the normalized matrix out of [-1, 1], which the check phase's bound takes
    for granted: it then goes on until the largest pair of the rest has converged."""
    (rp, c, v, n0), _ = wl.stochastic_block_model(1200, 10, 0.33, 0.002, 3)
    n, k = n0 + 2, 11
    w = np.zeros((n, n))
    for i in range(n0):
        w[i, c[rp[i]:rp[i + 1]]] = v[rp[i]:rp[i + 1]]
    w[n0, n0 + 1] = w[n0 + 1, n0] = 50.0         # +-1.001 with the two weights below zero
    w[n0, 0] = w[0, n0] = w[n0 + 1, 700] = w[700, n0 + 1] = -0.05
    rows, cols = np.nonzero(w)
    rp = np.searchsorted(rows, np.arange(n + 1)).astype(np.int64)
    g = (rp, cols.astype(np.int32), w[rows, cols], n)
    s = 1.0 / np.sqrt(w.sum(1))
    lam0 = 1.0 - np.linalg.eigvalsh(s[:, None] * w * s[None, :])[::-1]
    assert lam0[0] < -1e-4 and lam0[-1] > 2.0 + 1e-4 and lam0[k] - lam0[k - 1] > 0.2
    lam, vec, code, stats = solve(B, g, k, 1e-10, block=block, m=96)
    assert code == B.SC_OK
    assert np.max(np.abs(lam - lam0[:k])) <= 1e-9
    assert np.max(compare.residual_norms(*g[:3], lam, vec)) <= 1e-8
    _, _, _, locking = solve(B, g, k, 1e-10, block=block, m=96, flags=B.SC_FLAG_NO_VERIFY)
    # the rest's spectrum is dense at its upper end: nothing there converges in a few steps
    steps = stats["block_steps"] - locking["block_steps"]
    assert steps >= 15, steps


# Steps and block QRs as one launch.  Rows on either side of a workgroup's share and of the most that 128 workgroups take; with
# m = 300 and no filter a basis that outgrows the workgroups' LDS (128 columns of 128 rows); a row too long for a lane group (whose
# QRs are taken that way all the same); blocks of 16, whose QRs alone are, up to the rows that 256 workgroups hold.
@pytest.mark.parametrize("n,k,m,block,way", [(60, 3, 0, 8, "all"), (65, 4, 0, 8, "all"), (129, 6, 0, 8, "all"), (2000, 9, 0, 8, "all"),
                                             (4033, 10, 0, 8, "all"), (8192, 12, 0, 8, "all"), (8193, 12, 300, 8, "some"),
                                             (16384, 8, 0, 8, "all"), (16385, 8, 0, 8, "qr"), (2000, 9, 0, 8, "hub"),
                                             (100, 5, 0, 16, "qr"), (16385, 20, 0, 16, "qr"), (100_003, 20, 0, 16, "qr"),
                                             (240_000, 4, 0, 16, "qr"), (300_000, 4, 0, 16, "none"), (2000, 9, 0, 4, "none")])
def test_block_step_as_one_launch(B, monkeypatch, n, k, m, block, way):
    """Launches whose workgroups exchange sums, the ordinary launches, and a solve whose first such launch finds that its workgroups
    cannot all have started: the same pairs."""
    rp, c, v, n = wl.random_weighted_connected(n, 4 * n, 5 + n)
    if way == "hub":  # node 0 is tied to 200 others
        rp, c, v, n = wl.disjoint_union((rp, c, v, n), wl.complete_bipartite(1, 200))
    g = (rp, c, v, n)
    flags = B.SC_FLAG_NO_START_FILTER if way == "some" else 0
    runs = []
    for env in ({}, {"SCEIG_NO_FUSED": "1"}, {"SCEIG_FUSED_POLLS": "-1"}):
        for name, value in env.items():
            monkeypatch.setenv(name, value)
        before = [B.sc_counter(x) for x in (B.SC_COUNTER_FUSED_STEPS, B.SC_COUNTER_FUSED_QRS)]
        lam, vec, code, stats = solve(B, g, k, 1e-9, block=block, m=m, flags=flags)
        steps, qrs = [B.sc_counter(x) - y for x, y in zip((B.SC_COUNTER_FUSED_STEPS, B.SC_COUNTER_FUSED_QRS), before)]
        for name in env:
            monkeypatch.delenv(name)
        assert code == B.SC_OK, stats
        if env or way == "none":
            assert steps == 0 and qrs == 0, (env, steps, qrs)
        else:
            assert qrs > 0
            assert {"all": steps == stats["block_steps"], "some": 0 < steps < stats["block_steps"]}.get(way, steps == 0), (steps, stats)
        assert compare.residual_norms(rp, c, v, lam, vec).max() <= 1e-8
        assert compare.orthonormality_defect(vec) <= 1e-12
        runs.append(lam)
    assert np.max(np.abs(runs[0] - runs[1])) <= 1e-11 and np.max(np.abs(runs[2] - runs[1])) <= 1e-11


# The way back in the middle of a solve: the workgroups of launch number `stop` (the start block's QR is the first) find that they
# cannot all start, and with them those of all further ones.  A step, one that had the next one enqueued behind it, and that one;
# QRs behind ordinary launches (blocks of 16); bases that outgrow the workgroups' LDS, with restarts; blocks of several phases.
@pytest.mark.parametrize("graph,k,m,block,flags,stops", [("random", 9, 0, 8, 0, (2, 3, 4, 5, 8, 13, 21, 40)),
                                                         ("wide", 12, 300, 8, "nofilter", (2, 7, 12, 17, 18, 30)),
                                                         ("narrow", 9, 40, 8, "nofilter", (3, 6, 9, 11, 20, 60)),
                                                         ("comps", 30, 0, 8, 0, (2, 3, 6, 7, 10, 12)),
                                                         ("random16", 20, 0, 16, 0, (2, 3, 5, 9)),
                                                         ("comps16", 40, 0, 16, 0, (2, 3, 4, 5))])
def test_fused_launches_that_stop_in_the_middle(B, monkeypatch, graph, k, m, block, flags, stops):
    if graph.startswith("comps"):
        rp, c, v, n = wl.disjoint_union(*[wl.random_weighted_connected(60 + 7 * t, 200, t) for t in range(k)])
    else:
        n = {"random": 2000, "wide": 8193, "narrow": 3000, "random16": 16385}[graph]
        rp, c, v, n = wl.random_weighted_connected(n, 4 * n, 5 + n)
    g = (rp, c, v, n)
    flags = B.SC_FLAG_NO_START_FILTER if flags == "nofilter" else 0

    def run(**env):
        for name, value in env.items():
            monkeypatch.setenv(name, value)
        before = [B.sc_counter(x) for x in (B.SC_COUNTER_FUSED_STEPS, B.SC_COUNTER_FUSED_QRS)]
        lam, vec, code, stats = solve(B, g, k, 1e-9, block=block, m=m, flags=flags)
        ran = sum(B.sc_counter(x) - y for x, y in zip((B.SC_COUNTER_FUSED_STEPS, B.SC_COUNTER_FUSED_QRS), before))
        for name in env:
            monkeypatch.delenv(name)
        assert code == B.SC_OK, (env, stats)
        assert compare.residual_norms(rp, c, v, lam, vec).max() <= 1e-8, env
        assert compare.orthonormality_defect(vec) <= 1e-12, env
        return lam, ran

    plain, ran = run(SCEIG_NO_FUSED="1")
    assert ran == 0
    lam, whole = run()
    assert np.max(np.abs(lam - plain)) <= 1e-11
    stopped = 0
    for stop in stops:
        lam, ran = run(SCEIG_FUSED_STOP=str(stop))
        assert ran <= stop - 1 and (ran > 0 or stop == 1), (stop, ran, whole)  # a step that was not asked for is none of them
        stopped += ran < whole
        assert np.max(np.abs(lam - plain)) <= 1e-11, stop
    assert stopped >= 2, whole


def test_steps_that_were_not_asked_for_are_not_timed(B):
    """One-launch steps are timed with the reductions, of which a phase without locked vectors has none; the one that a solve has
    enqueued ahead of its last inspection belongs to no step."""
    rp, c, v, n = wl.random_weighted_connected(2000, 8000, 11)
    before = B.sc_counter(B.SC_COUNTER_FUSED_STEPS)
    _, _, code, stats = solve(B, (rp, c, v, n), 4, 1e-9, block=8, flags=B.SC_FLAG_NO_VERIFY, timing_mask=63)
    assert code == B.SC_OK and stats["phases"] == 1
    assert B.sc_counter(B.SC_COUNTER_FUSED_STEPS) - before == stats["block_steps"] > 0
    assert stats["fam_launches"][5] == stats["block_steps"], stats
    assert stats["fam_time_s"][5] > 0.0 and stats["fam_flops"][5] > 0.0


# Two callers at once, whose one-launch forms take the compute units from one another (a workgroup of these QRs fills the LDS), so
# that which of them start is settled on the device: the same results, but for the last bits.
@pytest.mark.parametrize("n,b,nodes,k,block", [(557_056, 8, 2000, 9, 8), (94_208, 32, 4033, 10, 8), (258_048, 16, 16385, 20, 16)])
def test_fused_launches_of_two_callers(B, n, b, nodes, k, block):
    import threading
    rp, c, v, _ = wl.random_weighted_connected(nodes, 4 * nodes, 5 + nodes)
    dev = B.csr_to_device(rp, c, v)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    start = torch.randn((n, b), dtype=torch.float64, generator=gen, device="cuda")
    alone = start.clone()
    B.sc_block_qr(alone, 0, b)
    lam0 = B.sc_laplacian_eigsh(*dev, k, 1e-9, block=block)[0]
    torch.cuda.synchronize()
    eye = torch.eye(b, dtype=torch.float64, device="cuda")
    wrong = []

    def call(first):
        with torch.cuda.stream(torch.cuda.Stream()):
            for r in range(12):
                if (r + first) % 3 != 2:
                    basis = start.clone()
                    B.sc_block_qr(basis, 0, b)
                    if (basis.T.contiguous() @ basis - eye).abs().max() > 1e-13 or (basis - alone).abs().max() > 1e-10:
                        wrong.append(("qr", first, r))
                else:
                    lam, _, code, _ = B.sc_laplacian_eigsh(*dev, k, 1e-9, block=block)
                    if code != B.SC_OK or (lam - lam0).abs().max() > 1e-11:
                        wrong.append(("solve", first, r))
        wrong.append(first)

    callers = [threading.Thread(target=call, args=(t,)) for t in range(2)]
    for t in callers:
        t.start()
    for t in callers:
        t.join()
    assert sorted(wrong, key=str) == [0, 1], wrong


# more components among the nodes that a workgroup counts than its table has places, beside some too large for most work items
@pytest.mark.parametrize("tiny,large", [(9000, (1500, 2000)), (700, (1273,)), (3000, ())])
def test_component_sizes_of_many_components(B, tiny, large):
    g = wl.disjoint_union(*[wl.random_weighted_connected(m, 4 * m, 3) for m in large], *[wl.complete(3)] * tiny)
    perm = np.random.default_rng(tiny).permutation(g[3])
    g = wl.relabel(g, perm)
    rp, c, v, n = g
    lam, vec, code, stats = solve(B, g, 20, 1e-9, block=16)
    assert code == B.SC_OK and stats["components"] == tiny + len(large)
    assert np.max(np.abs(lam)) <= 1e-9
    assert compare.residual_norms(rp, c, v, lam, vec).max() <= 1e-8
    assert compare.orthonormality_defect(vec) <= 1e-10


# the filter's items as pinned words and, beyond 65,536 of them, as pageable ones (five an item, an item or more a block)
@pytest.mark.parametrize("blocks", [3000, 13_107, 13_108, 70_000])
def test_filter_items_of_many_blocks(B, blocks):
    n = 3 * blocks
    rp = np.arange(0, 6 * blocks + 1, 2, dtype=np.int64)
    row = np.repeat(np.arange(n), 2).reshape(n, 2)
    c = (row // 3 * 3 + (row + [[1, 2]] - row // 3 * 3) % 3).astype(np.int32)
    c.sort(axis=1)
    before = B.sc_counter(B.SC_COUNTER_RESIDENT_FILTERS)
    lam, vec, code, stats = solve(B, (rp, c.reshape(-1), np.ones(6 * blocks), n), 40, 1e-9, block=16)
    assert code == B.SC_OK and stats["components"] == blocks
    assert B.sc_counter(B.SC_COUNTER_RESIDENT_FILTERS) > before
    assert np.max(np.abs(lam)) <= 1e-9
    assert compare.residual_norms(rp, c.reshape(-1), np.ones(6 * blocks), lam, vec).max() <= 1e-8
    assert compare.orthonormality_defect(vec) <= 1e-10


# labels that need more rounds than are made before the numbering goes on unseen (a path in random order), and more nodes than that
# is done for
@pytest.mark.parametrize("n", [3000, 60_000, 200_000, 200_001])
def test_renumbering_of_components_that_settle_late(B, n):
    parts = [wl.path(n // 2), wl.ring(n // 3), wl.path(n - n // 2 - n // 3)]
    g = wl.relabel(wl.disjoint_union(*parts), np.random.default_rng(n).permutation(n))
    rp, c, v, n = g
    comp = components.component_labels(rp, c, v)[1]
    drp, dc, dv = B.csr_to_device(rp, c, v)
    rpo, co, vo, old, count = B.sc_reorder_csr(drp, dc, dv)
    assert count == 3
    old = old.cpu().numpy()
    assert np.array_equal(np.sort(old), np.arange(n)) and np.count_nonzero(np.diff(comp[old])) == 2
    inverse = np.empty(n, dtype=np.int64)
    inverse[old] = np.arange(n)
    rpo, co = rpo.cpu().numpy(), co.cpu().numpy()
    row = np.repeat(np.arange(n), np.diff(rp))
    want = np.sort(inverse[row] * n + inverse[np.asarray(c)])
    assert np.array_equal(np.sort(np.repeat(np.arange(n), np.diff(rpo)) * np.int64(n) + co), want)
