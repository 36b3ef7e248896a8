"""What is measured: the calls a spectral-clustering program makes, through the public entry points of the binding.

The stages are those of the pipeline: neighbour graph from points, similarity graph from a pair list, eigensolve, the
eigensolver's steps for programs that drive their own iteration (product, block step, rotation), k-means.  Sizes are
those of the repository's workloads (config 1, 2 and 5 of `workloads.CONFIGS`, half of config 3, the FB- and DTI-shaped
inputs), some moved to odd ones.  Inputs are made on the GPU from the seed alone; everything is fp64, the only type the
library takes.

The mixture graphs take every point's neighbours inside its own component: the centres of the workloads lie so far apart
that this is the neighbour graph of the whole set.  Their k smallest eigenpairs (k = number of components) are the null
space, a basis of which is arbitrary, so those cases return what a program reads off the row-normalised embedding: the
cosine of every node with some query nodes.  It does not depend on the basis, and is 1 inside a component and 0 outside.
"""
import math

import numpy as np
import torch

from paper_1802_04450_amd import binding as sc

DEV = "cuda:0"


# ---- cases ------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # eigensolve of a small graph, all latency (config 1)
        dict(name="eigsh_2k", kind="eigsh", n=2000, comps=8, d=16, k_nn=10, weights="equal", std=1.0, tol=1e-10,
             own=False),
        # the ordinary eigensolve: hubs, components of very different sizes (config 2)
        dict(name="eigsh_100k", kind="eigsh", n=100_000, comps=100, d=32, k_nn=20, weights="dirichlet", std=1.5, tol=1e-8,
             own=False),
        # many vertices, components of which a part is too large for a compute unit (half of config 3)
        dict(name="eigsh_500k_k500", kind="eigsh", n=500_000, comps=500, d=64, k_nn=16, weights="dirichlet", std=1.5,
             tol=1e-8, own=False),
        # the largest: many eigenvectors (config 5), in a workspace that the program owns
        dict(name="eigsh_500k_k2000", kind="eigsh", n=500_000, comps=2000, d=128, k_nn=10, weights="equal", std=1.0,
             tol=1e-7, own=True),
        # a connected graph with simple eigenvalues (the FB-shaped block model): the eigenvectors themselves
        dict(name="eigsh_connected_4k", kind="connected", n=4040, comps=10, tol=1e-10),
        # the single-vector product of a program's own iteration, large and irregular
        dict(name="spmv_2m", kind="product", n=2_000_003, radius2=5, cols=1),
        # one block step of a program's own block Lanczos: product, reorthogonalization, block QR
        dict(name="step_100k_b16", kind="step", n=100_003, comps=100, d=32, k_nn=20, j=200, b=16),
        dict(name="step_500k_b32", kind="step", n=500_000, comps=2000, d=128, k_nn=10, j=992, b=32),
        # a thick restart: half of 400 Krylov vectors are kept
        dict(name="rotate_300k", kind="rotate", n=300_007, j0=16, ja=400, l=200, colmajor=False),
        # clustering of the embedding, in the layout that the eigensolver returns (config 2's shape)
        dict(name="kmeans_100k", kind="kmeans", n=100_000, d=100, k=100, colmajor=True),
        # similarity graph of the DTI shape: 142,541 voxels with 90 coordinates, pairs within 4 mm
        dict(name="similarity_142k", kind="similarity", n=142_541, d=90, radius2=5, measure=0),
        # neighbour graph of config 2's points
        dict(name="knn_100k", kind="knn", n=100_000, d=32, k_nn=20, comps=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eigsh", "eigsh", "eigsh", "connected", "product", "product", "step", "step", "rotate", "rotate",
                       "kmeans", "kmeans", "similarity", "similarity", "knn", "knn"])
    if kind == "eigsh":
        n = _log_int(rng, 2000, 400_000)
        size = _log_int(rng, 200, 2000)
        d = _log_int(rng, 16, 128)
        return dict(kind=kind, n=n, comps=max(4, min(1000, n // size)), d=d, k_nn=rng.randint(10, 20),
                    weights=rng.choice(["equal", "dirichlet"]), std=rng.choice([1.0, 1.5]), tol=rng.choice([1e-7, 1e-8, 1e-10]), own=rng.random() < 0.4)
    if kind == "connected":
        comps = rng.randint(4, 16)
        return dict(kind=kind, n=comps * _log_int(rng, 250, 750), comps=comps, tol=1e-10)
    if kind == "product":
        cols = rng.choice([1, 1, 1, 2, 4, 8, 16, 32])
        return dict(kind=kind, n=_log_int(rng, 2000, 2_000_000 // math.isqrt(cols)), radius2=rng.choice([1, 2, 3, 5, 6]), cols=cols)
    if kind == "step":
        n = _log_int(rng, 2000, 500_000)
        b = rng.choice([8, 16, 32])
        return dict(kind=kind, n=n, comps=max(4, n // _log_int(rng, 200, 1000)), d=_log_int(rng, 16, 128),
                    k_nn=rng.randint(10, 20), j=_log_int(rng, b, min(992, n // 4)), b=b)
    if kind == "rotate":
        n = _log_int(rng, 2000, 300_000)
        ja = _log_int(rng, 8, 400)
        return dict(kind=kind, n=n, j0=rng.randint(0, 40), ja=ja, l=rng.randint(1, ja), colmajor=rng.random() < 0.3)
    if kind == "kmeans":
        return dict(kind=kind, n=_log_int(rng, 2000, 140_000), d=_log_int(rng, 2, 128), k=_log_int(rng, 2, 128),
                    colmajor=rng.random() < 0.6)
    if kind == "similarity":
        return dict(kind=kind, n=_log_int(rng, 2000, 142_541), d=_log_int(rng, 8, 128), radius2=rng.choice([1, 2, 3, 5, 6]),
                    measure=rng.choice([0, 0, 1, 2]))
    n = _log_int(rng, 2000, 100_000)
    return dict(kind=kind, n=n, d=_log_int(rng, 3, 64), k_nn=_log_int(rng, 5, 32), comps=max(1, n // _log_int(rng, 500, 2000)))


# ---- inputs -----------------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 12345)
    return g


def _sizes(n, comps, weights, least, seed):
    rng = np.random.default_rng(int(seed) + 17)
    w = rng.dirichlet(np.full(comps, 5.0)) if weights == "dirichlet" else np.full(comps, 1.0 / comps)
    size = np.maximum(rng.multinomial(n, w), least)
    while size.sum() > n:
        big = int(size.argmax())
        size[big] -= min(size.sum() - n, max(1, size[big] // 8))
    size[int(size.argmin())] += n - size.sum()
    return size, rng


def _symmetric_csr(u, v, w, n):
    """CSR of the undirected edges (u, v, w), each listed once."""
    key = torch.cat([u * n + v, v * n + u])
    key, at = torch.sort(key)
    val = torch.cat([w, w])[at]
    row = torch.div(key, n, rounding_mode="floor")
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return rowptr, (key - row * n).to(torch.int32), val


def _mixture_graph(n, comps, d, k_nn, weights, std, seed):
    """Gaussian-weighted neighbour graph (union) of a Gaussian mixture, nodes in random order.  (rowptr, col, val, label)."""
    size, rng = _sizes(n, comps, weights, 2 * k_nn + 2, seed)
    scale = rng.uniform(0.5, 1.5, size=comps) if std != 1.0 else np.ones(comps)
    gen = _gen(seed)
    node = torch.randperm(n, generator=gen, device=DEV)
    us, vs, ds = [], [], []
    start = 0
    for c in range(comps):
        s = int(size[c])
        x = torch.randn((s, d), dtype=torch.float64, generator=gen, device=DEV) * float(scale[c])
        sq = (x * x).sum(1)
        d2 = sq[:, None] + sq[None, :] - 2.0 * (x @ x.T)
        d2.fill_diagonal_(float("inf"))
        near, at = torch.topk(d2, k_nn, dim=1, largest=False)
        own = node[start:start + s]
        us.append(own[:, None].expand(s, k_nn).reshape(-1))
        vs.append(own[at].reshape(-1))
        ds.append(near.reshape(-1))
        start += s
    u, v, d2 = torch.cat(us), torch.cat(vs), torch.cat(ds).clamp_(min=0.0)
    label = torch.empty(n, dtype=torch.int64, device=DEV)
    label[node] = torch.repeat_interleave(torch.arange(comps, device=DEV), torch.from_numpy(size).to(DEV))
    key, at = torch.sort(torch.minimum(u, v) * n + torch.maximum(u, v), stable=True)
    first = torch.ones(key.numel(), dtype=torch.bool, device=DEV)
    first[1:] = key[1:] != key[:-1]
    key, at = key[first], at[first]
    w = torch.exp(-d2[at] / (2.0 * d2.median()))
    lo = torch.div(key, n, rounding_mode="floor")
    return (*_symmetric_csr(lo, key - lo * n, w, n), label)


def _block_model(n, comps, seed):
    """Unit-weight block model, 40 edges a node inside its group and 2.2 between groups (the FB-shaped graph's densities)."""
    size = n // comps
    p, q = min(0.5, 40.0 / size), 2.2 / (n - size)
    gen = _gen(seed)
    us, vs = [], []
    for r0 in range(0, n, 2048):
        r = torch.arange(r0, min(n, r0 + 2048), device=DEV)[:, None]
        c = torch.arange(n, device=DEV)[None, :]
        same = torch.div(r, size, rounding_mode="floor") == torch.div(c, size, rounding_mode="floor")
        pick = torch.rand((r.numel(), n), generator=gen, device=DEV) < torch.where(same, p, q)
        # node i is always tied to the next one of its group, so that none is isolated
        pick |= same & (c == r + 1)
        at = torch.nonzero(pick & (c > r))
        us.append(at[:, 0] + r0)
        vs.append(at[:, 1])
    u, v = torch.cat(us), torch.cat(vs)
    return _symmetric_csr(u, v, torch.ones(u.numel(), dtype=torch.float64, device=DEV), n)


def _voxel_pairs(n, radius2):
    """Every pair of the first n cells of a cubic grid whose offset has squared length <= radius2, once, offset by offset.
    Yields (u, v, squared length)."""
    side = 1
    while side ** 3 < n:
        side += 1
    idx = torch.arange(n, dtype=torch.int64, device=DEV)
    ix, iy, iz = idx % side, torch.div(idx, side, rounding_mode="floor") % side, torch.div(idx, side * side, rounding_mode="floor")
    r = math.isqrt(radius2)
    for dz in range(0, r + 1):
        for dy in range(-r, r + 1):
            for dx in range(-r, r + 1):
                q = dx * dx + dy * dy + dz * dz
                if q > radius2 or (dz, dy, dx) <= (0, 0, 0):
                    continue
                j = idx + dx + dy * side + dz * side * side
                ok = (ix + dx >= 0) & (ix + dx < side) & (iy + dy >= 0) & (iy + dy < side) & (iz + dz < side) & (j < n)
                yield idx[ok], j[ok], q


def _voxel_graph(n, radius2, seed):
    """Voxel neighbourhood graph with a tenth of the longer edges missing, random weights, nodes in random order."""
    gen = _gen(seed)
    node = torch.randperm(n, generator=gen, device=DEV)
    us, vs, ws = [], [], []
    for u, v, q in _voxel_pairs(n, radius2):
        if q > 1:
            keep = torch.rand(u.numel(), generator=gen, device=DEV) < 0.9
            u, v = u[keep], v[keep]
        us.append(node[u])
        vs.append(node[v])
        ws.append(math.exp(-q / 4.0) * (0.5 + torch.rand(u.numel(), dtype=torch.float64, generator=gen, device=DEV)))
    return _symmetric_csr(torch.cat(us), torch.cat(vs), torch.cat(ws), n)


def _orthonormal(n, j, gen):
    q = torch.randn((n, j), dtype=torch.float64, generator=gen, device=DEV)
    return q @ torch.linalg.inv(torch.linalg.cholesky(q.T @ q)).mT


def _blobs(n, d, k, spread, gen):
    cen = torch.randn((k, d), dtype=torch.float64, generator=gen, device=DEV)
    lab = torch.randint(0, k, (n,), generator=gen, device=DEV)
    return cen[lab] + spread * torch.randn((n, d), dtype=torch.float64, generator=gen, device=DEV)


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    gen = _gen(seed + 1)
    if kind == "eigsh":
        rowptr, col, val, label = _mixture_graph(n, case["comps"], case["d"], case["k_nn"], case["weights"], case["std"], seed)
        query = torch.randint(0, n, (16,), generator=gen, device=DEV)
        room = sc.sc_workspace_bytes(n, col.numel(), case["comps"]) if case["own"] else 0
        return dict(kind=kind, rowptr=rowptr, col=col, val=val, k=case["comps"], tol=case["tol"], query=query, label=label,
                    workspace=torch.empty(room, dtype=torch.uint8, device=DEV) if case["own"] else None)
    if kind == "connected":
        rowptr, col, val = _block_model(n, case["comps"], seed)
        return dict(kind=kind, rowptr=rowptr, col=col, val=val, k=case["comps"], tol=case["tol"])
    if kind == "product":
        rowptr, col, val, _, _ = sc.sc_reorder_csr(*_voxel_graph(n, case["radius2"], seed))
        _, s = sc.sc_degree_scaling(rowptr, col, val, want_degrees=False)
        x = torch.randn((n, case["cols"]), dtype=torch.float64, generator=gen, device=DEV)
        st = dict(kind=kind, rowptr=rowptr, col=col, val=val, s=s, cols=case["cols"], y=torch.empty_like(x), work=torch.empty_like(x))
        if case["cols"] == 1:
            st.update(x=s * x[:, 0], y=torch.empty_like(s), work=torch.empty_like(s), nnz=col.numel())
        else:
            st.update(x=x)
        return st
    if kind == "step":
        graph = _mixture_graph(n, case["comps"], case["d"], case["k_nn"], "equal", 1.5, seed)
        rowptr, col, val, _, _ = sc.sc_reorder_csr(*graph[:3])
        _, s = sc.sc_degree_scaling(rowptr, col, val, want_degrees=False)
        j, b = case["j"], case["b"]
        basis = torch.zeros((n, (j + b + 15) // 16 * 16), dtype=torch.float64, device=DEV)
        basis[:, :j] = _orthonormal(n, j, gen)
        return dict(kind=kind, rowptr=rowptr, col=col, val=val, s=s, basis=basis, j=j, b=b,
                    work=torch.empty((n, b), dtype=torch.float64, device=DEV))
    if kind == "rotate":
        ld = (case["j0"] + case["ja"] + 31) // 16 * 16
        basis = torch.randn((n, ld), dtype=torch.float64, generator=gen, device=DEV) / math.sqrt(n)
        y = torch.linalg.qr(torch.randn((case["ja"], case["l"]), dtype=torch.float64, generator=gen, device=DEV))[0].contiguous()
        return dict(kind=kind, basis=basis, j0=case["j0"], ja=case["ja"], y=y, colmajor=case["colmajor"])
    if kind == "kmeans":
        x = _blobs(n, case["d"], case["k"], 0.15, gen)
        return dict(kind=kind, x=x.T.contiguous() if case["colmajor"] else x, k=case["k"], seed=int(seed) % 100_003,
                    colmajor=case["colmajor"])
    if kind == "similarity":
        pairs = list(_voxel_pairs(n, case["radius2"]))
        u = torch.cat([p[0] for p in pairs]).to(torch.int32)
        v = torch.cat([p[1] for p in pairs]).to(torch.int32)
        side = math.ceil(n ** (1.0 / 3.0))
        idx = torch.arange(n, device=DEV)
        pos = torch.stack([idx % side, torch.div(idx, side, rounding_mode="floor") % side,
                           torch.div(idx, side * side, rounding_mode="floor")], 1).double() / side
        freq = 0.5 + 2.5 * torch.rand((3, case["d"]), dtype=torch.float64, generator=gen, device=DEV)
        phase = 2 * math.pi * torch.rand(case["d"], dtype=torch.float64, generator=gen, device=DEV)
        x = torch.sin(2 * math.pi * (pos @ freq) + phase)
        x = (x + 0.3 * torch.randn((n, case["d"]), dtype=torch.float64, generator=gen, device=DEV)).abs()
        return dict(kind=kind, x=x, u=u, v=v, n=n, measure=case["measure"])
    # knn: points of a mixture in a box, in random order
    cen = 40.0 * torch.rand((case["comps"], case["d"]), dtype=torch.float64, generator=gen, device=DEV) - 20.0
    std = 0.5 + torch.rand(case["comps"], dtype=torch.float64, generator=gen, device=DEV)
    lab = torch.randint(0, case["comps"], (n,), generator=gen, device=DEV)
    x = cen[lab] + std[lab][:, None] * torch.randn((n, case["d"]), dtype=torch.float64, generator=gen, device=DEV)
    return dict(kind=kind, x=x, k_nn=case["k_nn"], n=n)


def _filled_up(rowptr, col, val, room):
    """The number of edges depends on the points: zeros up to the most there can be, so that all passes return one shape."""
    more = (0, room - col.numel())
    return {"rowptr": rowptr, "col": torch.nn.functional.pad(col, more), "val": torch.nn.functional.pad(val, more)}


# ---- one pass ---------------------------------------------------------------------------------------------------------
def run(st):
    kind = st["kind"]
    if kind == "eigsh":
        evals, evecs, _, _ = sc.sc_laplacian_eigsh(st["rowptr"], st["col"], st["val"], st["k"], st["tol"],
                                                   flags=sc.SC_FLAG_ROW_NORMALIZE, workspace=st["workspace"])
        return {"theta": 1.0 - evals, "cosine": evecs[:, st["query"]].T @ evecs}
    if kind == "connected":
        evals, evecs, _, _ = sc.sc_laplacian_eigsh(st["rowptr"], st["col"], st["val"], st["k"], st["tol"])
        top = torch.gather(evecs, 1, evecs.abs().argmax(1, keepdim=True))
        return {"evals": evals, "evecs": evecs * torch.sign(top)}      # signs as usual: the largest entry is positive
    if kind == "product":
        if st["cols"] == 1:
            sc.sc_spmv_normalized_chain(st["rowptr"], st["col"], st["val"], st["s"], st["nnz"], st["x"], st["y"], st["work"])
            return {"y": st["y"], "next": st["work"]}
        return {"y": sc.sc_spmm_normalized(st["rowptr"], st["col"], st["val"], st["s"], st["x"], y=st["y"], work=st["work"])}
    if kind == "step":
        basis, j, b = st["basis"], st["j"], st["b"]
        sc.sc_spmm_normalized(st["rowptr"], st["col"], st["val"], st["s"], basis[:, j - b:j], y=basis[:, j:j + b], work=st["work"])
        h = sc.sc_cgs2(basis, j, b)
        r, gram = sc.sc_block_qr(basis, j, b)
        return {"h": h, "r": r, "gram": gram, "block": basis[:, j:j + b]}
    if kind == "rotate":
        return sc.sc_rotate(st["basis"], st["j0"], st["ja"], st["y"], out_colmajor=st["colmajor"])
    if kind == "kmeans":
        labels, centres, _, stats = sc.sc_kmeans(st["x"], st["k"], st["seed"], max_iter=20, colmajor=st["colmajor"])
        return {"labels": labels, "centres": centres, "objective": stats["objective"]}
    if kind == "similarity":
        w = sc.sc_edge_similarity(st["x"], st["u"], st["v"], st["measure"])
        rowptr, col, val = sc.sc_coo_to_csr(st["u"], st["v"], w, st["n"], True)
        return {"pairs": w, "rowptr": rowptr, "col": col, "val": val}
    idx, dist = sc.sc_knn_search(st["x"], st["k_nn"])
    u, v, w = sc.sc_knn_union_pairs(idx, dist, float(dist.median()))
    return {"idx": idx, "dist": dist, **_filled_up(*sc.sc_coo_to_csr(u, v, w, st["n"], True), 2 * idx.numel())}


# ---- what a pass cannot do without ------------------------------------------------------------------------------------
def _graph_nnz(case):
    if case["kind"] == "product":
        return case["n"] * {1: 6, 2: 17, 3: 24, 5: 51, 6: 72}[case["radius2"]]
    return case["n"] * (42 if case["kind"] == "connected" else 1.6 * case["k_nn"])


def work(case):
    kind, n = case["kind"], case["n"]
    if kind in ("eigsh", "connected"):
        k, nnz = case["comps"], _graph_nnz(case)
        # the graph in, the vectors out; k vectors made orthonormal to one another, one product with each
        return {"bytes": 12 * nnz + 8 * (n + 1) + 8 * n * k, "flops": 2.0 * n * k * k + 2.0 * nnz * k}
    if kind == "product":
        nnz, b = _graph_nnz(case), case["cols"]
        return {"bytes": 12 * nnz + 16 * n + 8 * n * b * (3 if b == 1 else 2), "flops": 2.0 * nnz * b}
    if kind == "step":
        nnz, j, b = _graph_nnz(case), case["j"], case["b"]
        # the basis has to be read for the coefficients and again for the update, in each of the two passes
        return {"bytes": 12 * nnz + 16 * n + 4 * 8 * n * j + 8 * 8 * n * b, "flops": 2.0 * nnz * b + 8.0 * n * j * b + 8.0 * n * b * b}
    if kind == "rotate":
        return {"bytes": 8 * n * (case["ja"] + case["l"]) + 8 * case["ja"] * case["l"], "flops": 2.0 * n * case["ja"] * case["l"]}
    if kind == "kmeans":
        d, k = case["d"], case["k"]
        # a pass over the points for every seed, one labelling and one mean
        return {"bytes": 8 * n * d * (k + 1) + 4 * n + 8 * k * d, "flops": 3.0 * n * d * (k - 1) + 2.0 * n * d * k + n * d}
    if kind == "similarity":
        pairs = n * {1: 3, 2: 9, 3: 13, 5: 28, 6: 40}[case["radius2"]]
        return {"bytes": 8 * n * case["d"] + 16 * pairs + 24 * pairs + 8 * (n + 1), "flops": 2.0 * pairs * case["d"]}
    nnz = 1.6 * n * case["k_nn"]
    # a brute-force search forms every distance once for its two ends
    return {"bytes": 8 * n * case["d"] + 12 * n * case["k_nn"] + 12 * nnz + 8 * (n + 1), "flops": 1.0 * n * n * case["d"]}


def tolerance(case):
    kind = case["kind"]
    if kind == "eigsh":
        # a pair counts as converged at a residual of tol, and the gap behind the null space is 0.1 and more: vectors
        # of another path through the iteration are off by 10 tol at most (measured: 0.1 to 1 tol)
        return {"rel": 10 * case["tol"], "max": 1000 * case["tol"]}
    if kind == "connected":
        # gaps of 1e-3 between the eigenvalues of one cluster (measured: 3e-10)
        return {"rel": 1e3 * case["tol"], "max": 1e5 * case["tol"]}
    # four to ten times what the comparison with exact() shows
    return {"product": {"rel": 3e-15, "max": 3e-14}, "step": {"rel": 1e-13, "max": 1e-11}, "rotate": {"rel": 3e-15, "max": 3e-14},
            "kmeans": {"rel": 1e-14, "max": 1e-12, "differ": 1e-5}, "similarity": {"rel": 2e-15, "max": 2e-14},
            "knn": {"rel": 1e-15, "max": 1e-14}}[kind]


# ---- the same in plain 64-bit torch -----------------------------------------------------------------------------------
def _scaled(rowptr, col, val, n):
    row = torch.repeat_interleave(torch.arange(n, device=DEV), rowptr[1:] - rowptr[:-1])
    deg = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, row, val)
    s = deg.rsqrt()
    return row, s, s[row] * val * s[col.long()]


def _times(row, col, val, x):
    y = torch.zeros_like(x)
    step = max(1, 40_000_000 // x.shape[1])
    for e in range(0, val.numel(), step):
        y.index_add_(0, row[e:e + step], val[e:e + step, None] * x[col[e:e + step].long()])
    return y


def _draws(seed, k):
    """The counter-based numbers that sc_kmeanspp documents."""
    m = (1 << 64) - 1

    def mix(z):
        z = (z + 0x9E3779B97F4A7C15) & m
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
        return z ^ (z >> 31)

    return [(mix((mix(seed) + i) & m) >> 11) * 2.0 ** -53 for i in range(k)]


def _kmeans(x, k, seed, max_iter):
    n = x.shape[0]
    u = _draws(seed, k)
    at = int(u[0] * n)
    cen = [x[at]]
    d2 = ((x - x[at]) ** 2).sum(1)
    for i in range(1, k):
        run_sum = torch.cumsum(d2, 0)
        at = min(n - 1, int(torch.searchsorted(run_sum, (u[i] * run_sum[-1]).reshape(1), right=True)))
        cen.append(x[at])
        d2 = torch.minimum(d2, ((x - x[at]) ** 2).sum(1))
    cen = torch.stack(cen)
    labels = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    objective = -1.0
    for _ in range(max_iter):
        new = ((cen * cen).sum(1)[None, :] - 2.0 * (x @ cen.T)).argmin(1)
        if torch.equal(new, labels):
            objective = float(((x - cen[labels]) ** 2).sum())
            break
        labels = new
        count = torch.bincount(labels, minlength=k).double()[:, None]
        mean = torch.zeros_like(cen).index_add_(0, labels, x) / count.clamp(min=1.0)
        cen = torch.where(count > 0, mean, cen)
    return {"labels": labels.to(torch.int32), "centres": cen, "objective": objective}


def _to_csr(u, v, w, n):
    key = torch.cat([u.long() * n + v.long(), v.long() * n + u.long()])
    key, at = torch.sort(key, stable=True)
    row = torch.div(key, n, rounding_mode="floor")
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return {"rowptr": rowptr, "col": (key - row * n).to(torch.int32), "val": torch.cat([w, w])[at]}


def exact(case, seed):
    st, kind, n = prepare(case, seed), case["kind"], case["n"]
    if kind == "eigsh":
        same = st["label"][st["query"]][:, None] == st["label"][None, :]
        return {"theta": torch.ones(st["k"], dtype=torch.float64, device=DEV), "cosine": same.double()}
    if kind == "connected":
        if n > 6000:
            return None
        row, _, val = _scaled(st["rowptr"], st["col"], st["val"], n)
        dense = torch.zeros((n, n), dtype=torch.float64)
        dense[row.cpu(), st["col"].long().cpu()] = val.cpu()
        theta, vec = np.linalg.eigh(dense.numpy())
        vec = np.ascontiguousarray(vec[:, ::-1][:, :st["k"]].T)
        top = np.take_along_axis(vec, np.abs(vec).argmax(1)[:, None], 1)
        return {"evals": 1.0 - theta[::-1][:st["k"]].copy(), "evecs": vec * np.sign(top)}
    if kind == "product":
        row, s, val = _scaled(st["rowptr"], st["col"], st["val"], n)
        if case["cols"] > 1:
            return {"y": _times(row, st["col"], val, st["x"])}
        y = _times(row, st["col"], val, (st["x"] / s)[:, None])[:, 0]
        return {"y": y, "next": s * y}
    if kind == "step":
        row, s, val = _scaled(st["rowptr"], st["col"], st["val"], n)
        q = st["basis"][:, :st["j"]]
        w = _times(row, st["col"], val, q[:, -st["b"]:].contiguous())
        h1 = q.T @ w
        w = w - q @ h1
        h2 = q.T @ w
        w = w - q @ h2
        gram = w.T @ w
        r = torch.linalg.cholesky(gram).mT
        w = w @ torch.linalg.inv(r)
        r2 = torch.linalg.cholesky(w.T @ w).mT
        return {"h": h1 + h2, "r": r2 @ r, "gram": gram, "block": w @ torch.linalg.inv(r2)}
    if kind == "rotate":
        out = st["basis"][:, st["j0"]:st["j0"] + st["ja"]] @ st["y"]
        return out.T.contiguous() if st["colmajor"] else out
    if kind == "kmeans":
        return _kmeans(st["x"].T.contiguous() if st["colmajor"] else st["x"], st["k"], st["seed"], 20)
    if kind == "similarity":
        x, u, v = st["x"], st["u"].long(), st["v"].long()
        if case["measure"] == sc.SC_SIM_CROSS_CORRELATION:
            x = x - x.mean(1, keepdim=True)
        norm = x.norm(dim=1)
        w = torch.empty(u.numel(), dtype=torch.float64, device=DEV)
        for e in range(0, u.numel(), 1 << 20):
            a, b = u[e:e + (1 << 20)], v[e:e + (1 << 20)]
            w[e:e + (1 << 20)] = (torch.exp(-((x[a] - x[b]) ** 2).sum(1) / 2.0) if case["measure"] == sc.SC_SIM_EXP_DECAY
                                  else (x[a] * x[b]).sum(1) / (norm[a] * norm[b]))
        return {"pairs": w, **_to_csr(u, v, w, n)}
    x, k = st["x"], case["k_nn"]
    idx = torch.empty((n, k), dtype=torch.int64, device=DEV)
    dist = torch.empty((n, k), dtype=torch.float64, device=DEV)
    sq = (x * x).sum(1)
    for r0 in range(0, n, 2048):
        r1 = min(n, r0 + 2048)
        d2 = sq[r0:r1, None] + sq[None, :] - 2.0 * (x[r0:r1] @ x.T)
        d2[torch.arange(r1 - r0, device=DEV), torch.arange(r0, r1, device=DEV)] = float("inf")
        near = torch.topk(d2, min(n - 1, k + 8), dim=1, largest=False)[1].sort(1)[0]
        true = ((x[near] - x[r0:r1, None, :]) ** 2).sum(2).sqrt()
        true, at = torch.sort(true, dim=1, stable=True)
        dist[r0:r1], idx[r0:r1] = true[:, :k], torch.gather(near, 1, at)[:, :k]
    sigma = float(dist.median())
    u = torch.arange(n, device=DEV)[:, None].expand(n, k).reshape(-1)
    key, at = torch.sort(torch.minimum(u, idx.reshape(-1)) * n + torch.maximum(u, idx.reshape(-1)), stable=True)
    first = torch.ones(key.numel(), dtype=torch.bool, device=DEV)
    first[1:] = key[1:] != key[:-1]
    lo = torch.div(key[first], n, rounding_mode="floor")
    w = torch.exp(-dist.reshape(-1)[at[first]] ** 2 / (2.0 * sigma * sigma))
    return {"idx": idx.to(torch.int32), "dist": dist, **_filled_up(*_to_csr(lo, key[first] - lo * n, w, n).values(), 2 * n * k)}
