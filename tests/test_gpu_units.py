"""GPU test of the column-listed units of the wide-batch products on small dense
systems whose block edges can go wrong: one interface row up to several row
blocks, interiors of 1 to 33 rows, an interior without coupling, matrix entries
given in two pieces, and column counts around a multiple of 16.  Against a dense
FP64 solve; the systems have condition numbers below 100, so tolerance 1e-13
leaves a relative error below 1e-10 (FP64) and 1e-8 (mixed)."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def system(n_gamma, sizes, seed):
    """A = dense SPD over [interface | interiors], interiors coupled to the
    interface only (the second one not at all), every K_GG entry split in two."""
    rng = np.random.default_rng(seed)
    n = n_gamma + sum(sizes)
    A = np.zeros((n, n))
    blk = rng.uniform(-1, 1, (n_gamma, n_gamma))
    A[:n_gamma, :n_gamma] = blk + blk.T
    off = n_gamma
    for k, m in enumerate(sizes):
        s = slice(off, off + m)
        b = rng.uniform(-1, 1, (m, m))
        A[s, s] = b + b.T
        if k != 1:
            A[s, :n_gamma] = rng.uniform(-1, 1, (m, n_gamma)) * (rng.random((m, n_gamma)) < 0.4)
            A[:n_gamma, s] = A[s, :n_gamma].T
        off += m
    A[np.arange(n), np.arange(n)] = 1.1 * np.abs(A).sum(axis=1) + 1.0
    kgg = sp.csr_matrix(A[:n_gamma, :n_gamma])
    cut = rng.uniform(0.2, 0.8, kgg.nnz)
    order = np.repeat(np.arange(kgg.nnz), 2)                 # both pieces, one after the other
    val = np.empty(2 * kgg.nnz)
    val[0::2], val[1::2] = kgg.data * cut, kgg.data * (1.0 - cut)
    kgg2 = sp.csr_matrix(kgg.shape)
    kgg2.indptr, kgg2.indices, kgg2.data = 2 * kgg.indptr, kgg.indices[order], val
    p = workloads.DDProblem(n_dof=n, n_gamma=n_gamma, gamma_map=np.arange(n_gamma, dtype=np.int32), kgg=kgg2)
    off = n_gamma
    for m in sizes:
        s = slice(off, off + m)
        g = np.nonzero(np.abs(A[s, :n_gamma]).sum(axis=0))[0]
        p.i_maps.append(np.arange(off, off + m, dtype=np.int32))
        p.g_maps.append(g.astype(np.int32))
        p.kii.append(np.asfortranarray(A[s, s]))
        p.kig.append(sp.csr_matrix(A[s][:, g]))
        off += m
    return A, p


@pytest.mark.parametrize("n_gamma,sizes", [(1, (1, 2)), (15, (16, 3, 17)), (16, (5, 1)), (17, (33, 16, 1)),
                                           (100, (7, 20, 31))])
@pytest.mark.parametrize("nrhs", [8, 40])
@pytest.mark.parametrize("prec", [0, 1])
def test_units_of_ragged_blocks(n_gamma, sizes, nrhs, prec):
    import paper_2306_00094_amd as dd
    print(f"case units n_gamma={n_gamma} sizes={sizes} nrhs={nrhs} prec={prec}", flush=True)
    A, p = system(n_gamma, sizes, seed=n_gamma)
    b = np.random.default_rng(1).uniform(-1, 1, (nrhs, p.n_dof))
    ref = np.linalg.solve(A, b.T).T
    s = dd.Solver(p, max_nrhs=nrhs)
    s.factor(dd.DD_FP64)
    if prec == dd.DD_MIXED:
        s.factor(prec)                       # both factors: residual replacement
    for launch in (dd.DD_LAUNCH_KERNELS, dd.DD_LAUNCH_GRAPH):
        r = s.solve(torch.from_numpy(b).to("cuda"), prec=prec,
                    opts=dd.dd_default_opts(tol=1e-13, tiles=1, launch=launch))
        err = np.linalg.norm(r.u.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= (1e-10 if prec == dd.DD_FP64 else 1e-8)
    s.close()
