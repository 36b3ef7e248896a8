"""CPU-only checks of the boundary: the library loads, exports every symbol the header declares,
the host projected-eigenproblem solver is right, and argument errors that are decided before any
GPU work come back as error codes."""
import ctypes
import os
import re
import time

import numpy as np
import pytest

from paper_1802_04450_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "sceig.h")).read()
    declared = set(re.findall(r"\b(sc_[a-z0-9_]+)\s*\(", header))
    assert declared == set(binding.EXPORTS), declared ^ set(binding.EXPORTS)
    lib = binding.lib()
    for name in declared:
        assert hasattr(lib, name), name
    assert lib.sc_version() >= 100
    assert binding.strerror(binding.SC_EZERODEG)


def test_struct_layouts_match_header_sizes():
    # sc_options: 3 x int32 + uint32 + uint64 + uint32 + int32 + pointer = 40 bytes;
    # sc_stats: 8 x int32 + 2 x int64 + 4 x double + 3 x double[6] + int64[6] = 80 + 192 = 272
    assert ctypes.sizeof(binding.ScOptions) == 40
    assert ctypes.sizeof(binding.ScStats) == 272


@pytest.mark.parametrize("n", [1, 2, 3, 10, 57, 200])
def test_sym_eig_against_numpy(n):
    rng = np.random.default_rng(n)
    a = rng.standard_normal((n, n))
    a = a + a.T
    w, z = binding.sc_sym_eig(a)
    assert np.allclose(w, np.linalg.eigvalsh(a), atol=1e-11 * max(1, n))
    assert np.max(np.abs(z.T @ z - np.eye(n))) < 1e-11
    assert np.max(np.abs(a @ z - z * w[None, :])) < 1e-10 * max(1, n)


def test_sym_eig_structured_cases():
    # diagonal, repeated eigenvalues, block-tridiagonal with an arrow head and a decoupled -2 "ghost"
    w, z = binding.sc_sym_eig(np.diag([3.0, -1.0, 2.0, 2.0]))
    assert np.allclose(w, [-1.0, 2.0, 2.0, 3.0])
    n = 24
    t = np.zeros((n, n))
    t[np.arange(8), np.arange(8)] = np.linspace(1.0, 0.9, 8)
    rng = np.random.default_rng(0)
    c = 1e-3 * rng.standard_normal((4, 8))
    t[8:12, :8] = c
    t[:8, 8:12] = c.T
    for blk in range(8, n, 4):
        a = rng.standard_normal((4, 4))
        t[blk:blk + 4, blk:blk + 4] = 0.1 * (a + a.T)
        if blk + 4 < n:
            r = np.triu(rng.standard_normal((4, 4)))
            t[blk + 4:blk + 8, blk:blk + 4] = r
            t[blk:blk + 4, blk + 4:blk + 8] = r.T
    t[5, :] = 0.0
    t[:, 5] = 0.0
    t[5, 5] = -2.0
    w, z = binding.sc_sym_eig(t)
    assert np.allclose(w, np.linalg.eigvalsh(t), atol=1e-12)
    assert np.max(np.abs(t @ z - z * w[None, :])) < 1e-12
    ghost = np.argmin(np.abs(w + 2.0))
    assert abs(abs(z[5, ghost]) - 1.0) < 1e-14      # the decoupled row keeps its own unit eigenvector
    w_only, none = binding.sc_sym_eig(t, vectors=False)
    assert none is None and np.allclose(w_only, w, atol=1e-12)


def test_sym_eig_larger_parallel_path():
    n = 400
    rng = np.random.default_rng(1)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = np.concatenate([np.ones(40), rng.uniform(-1, 0.5, n - 40)])   # a 40-fold eigenvalue
    a = (q * lam) @ q.T
    w, z = binding.sc_sym_eig(a)
    assert np.allclose(w, np.sort(lam), atol=1e-11)
    assert np.max(np.abs(z.T @ z - np.eye(n))) < 1e-11
    assert np.max(np.abs(a @ z - z * w[None, :])) < 1e-11


@pytest.mark.parametrize("n,count", [(1, 1), (2, 2), (9, 3), (64, 16), (150, 75), (333, 40)])
def test_sym_eig_top_selected_vectors(n, count):
    rng = np.random.default_rng(n * 7 + count)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = rng.uniform(-1, 0.6, n)
    lam[: min(n, 12)] = 1.0 - 1e-15 * np.arange(min(n, 12))          # a tight cluster at the top, as in the solver
    a = (q * lam) @ q.T
    a = 0.5 * (a + a.T)
    w, z = binding.sc_sym_eig_top(a, count)
    assert np.allclose(w, np.linalg.eigvalsh(a), atol=1e-12)
    assert z.shape == (n, count)
    assert np.max(np.abs(z.T @ z - np.eye(count))) < 1e-12
    top = w[::-1][:count]
    assert np.max(np.abs(a @ z - z * top[None, :])) < 1e-12
    w_full, z_full = binding.sc_sym_eig(a)
    assert np.allclose(w, w_full, atol=1e-13)


def test_argument_errors_without_gpu():
    lib = binding.lib()
    one = ctypes.c_void_p(8)        # non-null dummy; never dereferenced because validation fails first
    null = ctypes.c_void_p(0)
    f = lib.sc_laplacian_eigsh
    assert f(null, one, one, 10, 2, 1e-8, 10, one, one, null, None, None) == binding.SC_EINVAL
    assert f(one, one, one, -1, 2, 1e-8, 10, one, one, null, None, None) == binding.SC_EINVAL
    assert f(one, one, one, 10, 0, 1e-8, 10, one, one, null, None, None) == binding.SC_EDOMAIN
    assert f(one, one, one, 10, 10, 1e-8, 10, one, one, null, None, None) == binding.SC_EDOMAIN   # k >= n
    assert f(one, one, one, 10, 2, -1.0, 10, one, one, null, None, None) == binding.SC_EDOMAIN
    assert f(one, one, one, 10, 2, float("nan"), 10, one, one, null, None, None) == binding.SC_EDOMAIN
    assert f(one, one, one, 10, 2, 1e-8, 0, one, one, null, None, None) == binding.SC_EDOMAIN      # maxiter < 1
    opt = binding.ScOptions(m=11)                                                                  # m > n
    assert f(one, one, one, 10, 2, 1e-8, 10, one, one, null, ctypes.byref(opt), None) == binding.SC_EDOMAIN
    opt = binding.ScOptions(m=10, block=3)                                                         # block not a power of 2
    assert f(one, one, one, 10, 2, 1e-8, 10, one, one, null, ctypes.byref(opt), None) == binding.SC_EDOMAIN
    opt = binding.ScOptions(m=10, block=4)                                                         # k + 3b > m
    assert f(one, one, one, 10, 2, 1e-8, 10, one, one, null, ctypes.byref(opt), None) == binding.SC_EDOMAIN
    assert lib.sc_spmm_normalized(one, one, one, one, 10, one, 3, one, 3, 3, null, null) == binding.SC_EDOMAIN
    assert lib.sc_spmm_normalized(one, one, one, one, 10, one, 2, one, 4, 4, null, null) == binding.SC_EDOMAIN  # ldx < ncols
    assert lib.sc_cgs2(null, 10, 8, 2, 2, null, null, null) == binding.SC_EINVAL
    assert lib.sc_cgs2(one, 10, 3, 2, 2, null, null, null) == binding.SC_EDOMAIN                         # ld < j + b
    assert lib.sc_block_qr(one, 10, 8, 2, 5, null, null, null) == binding.SC_EDOMAIN
    assert lib.sc_rotate(one, 10, 8, 0, 9, one, 2, one, 2, 0, null) == binding.SC_EDOMAIN          # ld < j0 + ja
    assert lib.sc_sym_eig(null, 3, one, null) == binding.SC_EINVAL
    assert lib.sc_sym_eig_top(one, 3, 4, one, one) == binding.SC_EDOMAIN
    assert lib.sc_sym_eig_top(one, 3, 2, one, null) == binding.SC_EINVAL
    assert lib.sc_degree_scaling(one, one, one, 0, null, one, null) == binding.SC_OK               # n = 0: nothing to do


def test_workspace_bytes_query():
    """Host-only query: the figure contains the big blocks (basis n x (m + b), rotation workspace, operator copy),
    grows with m, and fails exactly where a solve would."""
    from paper_1802_04450_amd import binding as B
    n, nnz, k = 500_000, 8_100_000, 2000
    w = B.sc_workspace_bytes(n, nnz, k, m=4000)
    basis = n * 4032 * 8                       # block 32 by default at this size: ld = roundup16(4000 + 32)
    rot = n * (4000 // 2 + 32) * 8
    copy = nnz * 12 + nnz * 8
    assert basis + rot + copy < w < 1.1 * (basis + rot + copy) + (64 << 20)
    assert B.sc_workspace_bytes(n, nnz, k, m=5000) > w
    assert B.sc_workspace_bytes(n, nnz, k, m=4000, flags=B.SC_FLAG_NO_REORDER) < w
    small = B.sc_workspace_bytes(2000, 30000, 8)
    assert 2000 * 64 * 8 < small < (64 << 20)    # dominated by the fixed partial-sum buffers at this size
    for bad in (dict(n=10, nnz=20, k=10), dict(n=10, nnz=20, k=0), dict(n=100, nnz=500, k=5, m=6),
                dict(n=100, nnz=500, k=5, m=101), dict(n=100, nnz=500, k=5, block=3)):
        with pytest.raises(B.ScError) as e:
            B.sc_workspace_bytes(**bad)
        assert e.value.code == B.SC_EDOMAIN
    assert B.lib().sc_workspace_bytes(100, 500, 5, None, None) == B.SC_EINVAL


def _size_query(name, *types):
    """A host-only scratch-size function of the library's kernels.h (C++ name)."""
    f = getattr(binding.lib(), name)
    f.restype, f.argtypes = ctypes.c_size_t, list(types)
    return f


def test_edge_similarity_scratch_is_in_proportion_to_the_pairs():
    f = _size_query("_ZN5sceig22edge_buckets_workspaceElil", ctypes.c_int64, ctypes.c_int32, ctypes.c_int64)
    used = 0
    for n in (13_158, 60_000, 142_541, 500_000, 1_000_003, 4_000_000):
        for d in (2, 5, 17, 90, 128, 380, 381):
            for per_row in (8, 9, 27, 40, 200):
                ne = n * per_row + 1
                need = f(n, d, ne)
                used += need > 0
                assert need <= 100 * ne + 2 ** 26 + 2 ** 17, (n, d, ne, need)
    assert used > 20


def test_coo_to_csr_scratch_is_in_proportion_to_the_entries():
    f = _size_query("_ZN5sceig20coo_to_csr_workspaceElli", ctypes.c_int64, ctypes.c_int64, ctypes.c_int32)
    for n in (1, 300, 4099, 70_001, 1_000_000, 8_000_000, 16_000_000):
        for total in (1, 1000, 100_000, 500_000, 2_200_000, 8_000_000, 33_000_000):
            if total > 256 * n or (n > 1_000_000 and total < 2_000_000):
                continue                        # the radix sort, whose own scratch takes a device to ask for
            assert f(total, n, 0) <= 100 * total + 2 ** 26 + 2 ** 18, (n, total)


def test_knn_screen_scratch_is_what_the_header_says():
    f = _size_query("_ZN5sceig20knn_screen_workspaceElii", ctypes.c_int64, ctypes.c_int32, ctypes.c_int32)
    for n in (100, 512, 5000, 60_000, 100_000, 2_000_000, 20_000_000, 400_000_000):
        for d in (1, 3, 8, 9, 16, 17, 32, 64, 100, 128, 129):
            dp = next((p for p in (8, 16, 32, 64, 128) if d <= p), (d + 7) // 8 * 8)
            for k in (1, 10, 60, 200):
                need = f(n, d, k)
                assert need <= n * (4 * max(dp, 16) + 34) + 2 ** 28 + 2 ** 20, (n, d, k, need)
                assert need == 0 or (d <= 128 and n >= 512)


def test_knn_group_scratch_is_what_the_header_says():
    f = _size_query("_ZN5sceig19knn_group_workspaceElii", ctypes.c_int64, ctypes.c_int32, ctypes.c_int32)
    for n in (512, 20_000, 45_000, 62_000, 100_000, 2_000_000, 20_000_000, 400_000_000):
        for d in (1, 8, 9, 17, 32, 100, 128, 129):
            dp = next((p for p in (8, 16, 32, 64, 128) if d <= p), (d + 7) // 8 * 8)
            for k in (1, 10, 60, 200):
                need = f(n, d, k)
                assert need <= n * (7 * max(dp, 16) + 40) + 2 ** 30 + 2 ** 28 + 2 ** 21, (n, d, k, need)
                assert need == 0 or (d <= 128 and n * n * max(dp, 16) >= 6e10)
    assert f(100_000, 32, 20) > 0


def test_label_screen_scratch_is_what_the_header_says():
    f = _size_query("_ZN5sceig22label_screen_workspaceElli", ctypes.c_int64, ctypes.c_int64, ctypes.c_int32)
    used = 0
    for n in (2_000, 50_000, 100_000, 500_000, 8_000_000):
        for d in (1, 4, 31, 32, 100, 128, 129, 500, 2000):
            for k in (1, 2, 64, 65, 100, 2000):
                ldx = (d + 3) // 4 * 4          # as the points are staged, and what the header counts by
                need = f(n, ldx, k)
                used += need > 0
                assert need <= 4 * (n + k + 64) * (d + 16) + 12 * n + 2100 * (d + 4) + 2 ** 20, (n, d, k, need)
                assert (need > 0) == (n * ldx * k >= 4e8)
    assert used > 20


def _items_model(starts, counts, b, nnz, steps=100.0, lds=162_816):
    f = binding.lib()._ZN5sceig20resident_items_modelEPKiS1_iildlPl
    f.restype = ctypes.c_double
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_int64, ctypes.c_double,
                  ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)]
    starts, counts, out = np.ascontiguousarray(starts, np.int32), np.ascontiguousarray(counts, np.int32), ctypes.c_int64(0)
    took = []
    for _ in range(3):
        t0 = time.perf_counter()
        step = f(starts.ctypes.data, counts.ctypes.data, len(starts) - 1, b, nnz, steps, lds, ctypes.byref(out))
        took.append(time.perf_counter() - t0)
    return step, out.value, min(took)


@pytest.mark.parametrize("sliced", [0, 1, 40])
def test_items_of_many_blocks_are_planned_once(sliced):
    """The host's part of the filter plan for 500,000 blocks whose entries fit the registers, alone and beside a few that need
    another form: it looks at the many once, not once per split and with a place in a queue each (0.3 s; 0.02 s)."""
    many, big = 500_000, 900
    rows = np.concatenate([np.full(many, 4), np.full(sliced, big)])
    starts = np.concatenate([[0], np.cumsum(rows)])
    # chunks beyond the first of rows of 3 and of 40 entries, extra rows, entries, these with their padding
    counts = np.concatenate([np.tile([0, 0, 0, 12, 64], (many, 1)),
                             np.tile([big, 2 * big, 0, 40 * big, 41 * big], (sliced, 1)).reshape(-1, 5)])
    nnz = int(counts[:, 3].sum())
    step, items, took = _items_model(starts, counts, 16, nnz)
    share = (many * 12 * 128.0 / 150e9 + sliced * 40 * big * 128.0 / 204e9) / 256
    assert share <= step <= share + 40 * big * 128.0 / 204e9 * (sliced > 0) + 4e-6
    assert many + sliced <= items <= many + 4 * sliced
    assert took < 0.13, took


@pytest.mark.parametrize("n,d,k,least,most", [
    (100_000, 100, 100, 3, 5), (500_000, 100, 128, 3, 4), (65_000, 64, 1000, 3, 3), (1_000_000, 8, 64, 4, 14), (200_000, 20, 100, 6, 25),
    (142_541, 500, 100, 3, 6), (20_000, 2000, 64, None, None), (5_000, 100, 1000, None, None), (40_000, 100, 100, None, None),
    (45_000, 16, 1000, None, None), (200_000, 2, 512, None, None), (10_000, 500, 256, None, None)])
def test_steps_that_bring_in_the_labelling_screen(n, d, k, least, most):
    """Around the measured numbers of labelling steps after which the reduced copy of the points has paid; never where a step
    by the screen takes longer than by the product."""
    f = binding.lib()._ZN5sceig18label_screen_stepsElli
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    steps = f(n, (d + 3) // 4 * 4, k)
    assert steps == 2 ** 31 - 1 if least is None else least <= steps <= most, steps


def test_items_of_equal_blocks_share_the_compute_units():
    """512 equal blocks: two for each of the 256 compute units, in either register form."""
    for b in (16, 32):
        starts = np.arange(513) * 100
        counts = np.tile([0, 0, 0, 1000, 1100], (512, 1))
        step, items, _ = _items_model(starts, counts, b, 512_000)
        assert items == 512 and step == pytest.approx(2 * 1000 * 8.0 * b / 150e9 + 1e-6, rel=1e-12)


def test_few_steps_do_not_bring_in_the_sliced_copy():
    """20 complete graphs of 1,000 nodes: a step by the sliced form takes a tenth less than by the product, and making the
    sliced copy as long as four of them."""
    starts = np.arange(21) * 1000
    counts = np.tile([999 * 31, 999 * 62, 999 * 15, 999_000, 64_000], (20, 1))
    nnz = 20 * 999_000
    general = 3e-6 + nnz * 128.0 / 14.5e12
    few, many = _items_model(starts, counts, 16, nnz, 24.0)[0], _items_model(starts, counts, 16, nnz, 600.0)[0]
    assert many < 0.95 * general < general < few
    assert few - many == pytest.approx((60e-6 + 37e-12 * nnz) * (1 / 24.0 - 1 / 600.0), rel=1e-9)


def test_no_plan_is_made_that_will_not_be_taken():
    """Sliced blocks whose padding is too much even in the narrowest slices, and blocks in registers that take longer than the
    general product: known from the counts, before anything is laid out."""
    starts = np.arange(101) * 900
    counts = np.tile([900, 1800, 0, 40 * 900, 41 * 900], (100, 1))
    step, items, _ = _items_model(starts, counts, 16, 100 * 40 * 900)
    assert step > 0 and items >= 100
    counts[:, 4] = 61 * 900
    step, _, _ = _items_model(starts, counts, 16, 100 * 40 * 900)
    assert step == -1.0
    # five blocks of 600 rows, 15 entries a row: 8 us a step for each, 3.4 by the product
    starts = np.arange(6) * 600
    counts = np.tile([0, 0, 0, 9000, 9600], (5, 1))
    step, _, _ = _items_model(starts, counts, 16, 5 * 9000)
    assert step == -1.0


def _chebyshev(y, degree, lo, hi):
    x = (2.0 * y - hi - lo) / (hi - lo)
    inside = np.cos(degree * np.arccos(np.clip(x, -1.0, 1.0)))
    return np.where(np.abs(x) <= 1.0, inside, np.cosh(degree * np.arccosh(np.maximum(np.abs(x), 1.0))))


def _undetected(theta, kappa, d, lo, a, steps, n, b):
    """log10 of the chance that an eigenvalue from kappa on stays below a largest Ritz value of theta: with P = T F, a share
    x of it in a column shows once x^2 P(kappa)^2 (kappa - theta) > max P^2 (theta + 1), the most that eigenvalues of
    [-1, theta] can pull the Rayleigh quotient of P(S) q below theta."""
    low, high = np.linspace(-1.0, theta, 6001), np.linspace(kappa, 1.0, 2001)
    f_low = np.abs(_chebyshev(low, d, lo, a)) if d else 1.0
    f_high = np.abs(_chebyshev(high, d, lo, a)) if d else 1.0
    best = 0.0
    for t in np.linspace(theta, kappa, 42)[1:-1]:
        most = np.max(f_low * np.abs(_chebyshev(low, steps - 1, -1.0, t)))
        least = np.min(f_high * np.abs(_chebyshev(high, steps - 1, -1.0, t)))
        share = most / max(least, 1e-300) * np.sqrt((theta + 1.0) / (kappa - theta))
        best = min(best, b * np.log10(share * np.sqrt(2.0 * n)))
    return best


def _check_steps_needed():
    f = binding.lib()._ZN5sceig18check_steps_neededEddiddli
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_double, ctypes.c_double, ctypes.c_int, ctypes.c_double, ctypes.c_double, ctypes.c_int64, ctypes.c_int]
    return f


@pytest.mark.parametrize("b", [1, 2, 8, 16, 32])
@pytest.mark.parametrize("theta,kappa,d,lo,a", [
    (0.5, 0.6, 0, -1.0, 0.0), (0.9, 0.999, 0, -1.0, 0.0), (-0.2, 0.3, 0, -1.0, 0.0), (0.98, 0.981, 0, -1.0, 0.0),
    (0.5, 0.6, 12, -1.0, 0.55), (0.5, 0.6, 40, -1.0, 0.53), (0.9, 0.93, 20, -0.4, 0.91), (0.9, 0.93, 6, -0.7, 0.6),
    (0.3, 0.95, 9, -1.0, 0.4), (0.99, 0.9999, 30, -0.5, 0.992)])
def test_check_phase_steps_leave_a_chance_of_1e_minus_20(b, theta, kappa, d, lo, a):
    """The number of block steps after which a solve stops looking for a larger eigenvalue, against the polynomials
    themselves: enough for what it promises, and not many more than that."""
    f = _check_steps_needed()
    for n in (50, 4040, 2_000_000):
        steps = f(theta, kappa, d, lo, a, n, b)
        assert 1 <= steps < 10_000
        assert _undetected(theta, kappa, d, lo, a, steps, n, b) <= -20.0
        fewer = int(0.8 * steps) - 2
        assert fewer < 1 or _undetected(theta, kappa, d, lo, a, fewer, n, b) > -20.0
        assert f(kappa, kappa, d, lo, a, n, b) == f(kappa + 0.001, kappa, d, lo, a, n, b) == 1 << 30


@pytest.mark.parametrize("b", [2, 8, 16, 32])
def test_check_phase_filter_that_makes_one_step_enough(b):
    """The shortest filters after which one block step is said to be enough: there is no room to spare in them."""
    f = _check_steps_needed()
    seen = 0
    for n in (60, 700, 4040, 100_003):
        for theta, kappa in ((0.5, 0.6), (0.9, 0.95), (0.97, 0.9999), (0.2, 0.7), (0.7, 0.73)):
            for part in (0.2, 0.4, 0.6):
                a = theta + part * (kappa - theta)
                d = next((q for q in range(2, 121) if f(theta + 0.05 * (kappa - theta), kappa, q, -1.0, a, n, b) == 1), None)
                if d is not None:
                    seen += 1
                    assert _undetected(theta + 0.05 * (kappa - theta), kappa, d, -1.0, a, 1, n, b) <= -20.0, (n, theta, kappa, a, d)
    assert seen >= 30


@pytest.mark.parametrize("b", [1, 8, 32])
@pytest.mark.parametrize("kappa", [0.55, 0.65, 0.7])
def test_check_phase_does_not_trust_a_filter_that_damps_what_it_asks_for(b, kappa):
    """A filter whose damped interval reaches past the value that something larger would have (a later phase has locked larger
    values than an earlier one) has zeros there: no number of steps shows an eigenvalue that it has put out."""
    f = _check_steps_needed()
    for d in (1, 2, 17, 30):
        assert f(0.5, kappa, d, -1.0, 0.7, 4040, b) == f(0.5, kappa, d, -0.4, 0.7, 4040, b) == 1 << 30
    assert f(0.5, kappa, 0, -1.0, 0.7, 4040, b) < 1000 and f(0.5, 0.701, 30, -1.0, 0.7, 4040, b) < 1000
