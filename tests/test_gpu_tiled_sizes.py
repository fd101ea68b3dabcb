"""GPU test of the tiled CG step where its reductions change with the interface:
slabs of 32, 64 and 128 rows (limits 8 192 and 32 768 rows), p^T q sums by row
blocks or by groups of them (limit 640 row blocks of 16), at 8 columns and more;
and of a row block whose column list does not fit the LDS of the kernel that fills
the units (4 096 columns).  Sparse systems with condition numbers below 100 against
a sparse FP64 solve: tolerance 1e-13 leaves a relative error below 1e-10 (FP64)
and 1e-8 (mixed, with and without residual replacement); the first columns have
equal bits at every width."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla

import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def system(n_gamma, sizes, wide_row=0, seed=0):
    """K_GG a band of five entries a row (and, for wide_row > 0, one row with that
    many more columns, and its mirror), dense interiors coupled to interface rows
    spread over the whole interface."""
    rng = np.random.default_rng(seed)
    n = n_gamma + sum(sizes)
    i = np.arange(n_gamma)
    r, c, v = [], [], []

    def add(rows, cols):
        x = rng.uniform(-1, 1, len(rows))
        r.extend([rows, cols])
        c.extend([cols, rows])
        v.extend([x, x])

    for d in (1, 2):
        add(i[:-d], i[d:])
    if wide_row:
        add(np.full(wide_row, 5), n_gamma - 1 - np.arange(wide_row))
    off = n_gamma
    for m in sizes:
        a = off + np.arange(m)
        x, y = np.triu_indices(m, 1)
        add(a[x], a[y])
        for t in range(3):
            add(a, rng.choice(n_gamma, m, replace=False))
        off += m
    A = sp.coo_matrix((np.concatenate(v), (np.concatenate(r), np.concatenate(c))), shape=(n, n)).tocsr()
    A = (A + sp.diags(1.1 * np.asarray(abs(A).sum(axis=1)).ravel() + 1.0)).tocsr()
    kgg = A[:n_gamma, :n_gamma].tocsr()
    kgg.sort_indices()
    p = workloads.DDProblem(n_dof=n, n_gamma=n_gamma, gamma_map=np.arange(n_gamma, dtype=np.int32), kgg=kgg)
    off = n_gamma
    for m in sizes:
        s = slice(off, off + m)
        kig = A[s, :n_gamma].tocsc()
        g = np.nonzero(np.diff(kig.indptr))[0]
        p.i_maps.append(np.arange(off, off + m, dtype=np.int32))
        p.g_maps.append(g.astype(np.int32))
        p.kii.append(np.asfortranarray(A[s, s].toarray()))
        p.kig.append(kig[:, g].tocsr())
        off += m
    return A, p


def check(n_gamma, sizes, prec, reliable, widths, wide_row=0):
    import paper_2306_00094_amd as dd
    A, p = system(n_gamma, sizes, wide_row)
    b = np.random.default_rng(1).uniform(-1, 1, (max(widths), p.n_dof))
    ref = spla.splu(A.tocsc()).solve(b.T).T
    s = dd.Solver(p, max_nrhs=max(widths))
    s.factor(dd.DD_FP64)
    if prec == dd.DD_MIXED:
        s.factor(prec)
    first = None
    for m in widths:
        print(f"case tiled n_gamma={n_gamma} wide={wide_row} prec={prec} reliable={reliable} columns={m}", flush=True)
        u = s.solve(torch.from_numpy(b[:m].copy()).cuda(), prec=prec,
                    opts=dd.dd_default_opts(tol=1e-13, tiles=1, reliable=reliable)).u.cpu().numpy()
        err = np.linalg.norm(u - ref[:m], axis=1) / np.linalg.norm(ref[:m], axis=1)
        assert err.max() <= (1e-10 if prec == dd.DD_FP64 else 1e-8), err
        first = u[:8] if first is None else first
        assert np.array_equal(u[:8], first), m
    s.close()


@pytest.mark.parametrize("n_gamma", [8191, 8192, 10240, 10241, 32767, 32768])
@pytest.mark.parametrize("prec,reliable", [(0, 0), (1, 0), (1, -1)])
def test_slabs_and_groups(n_gamma, prec, reliable):
    check(n_gamma, (40, 17, 33), prec, reliable, (8, 13, 32, 64))


@pytest.mark.parametrize("prec", [0, 1])
def test_wide_column_list(prec):
    check(6000, (70, 20), prec, 0, (8, 33), wide_row=4500)
