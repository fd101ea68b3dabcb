"""GPU test of the factorisation at the largest block of the one-launch Cholesky
(1 024 rows) and the first that goes panel by panel, alone and beside small blocks:
the factor against numpy's, the solution of a solve (a system with a condition
number below 100), and the column named when a block is not positive definite."""
import numpy as np
import pytest

from test_gpu_units import system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [(1024,), (1025,), (16, 1024, 5), (16, 1025, 5)])
@pytest.mark.parametrize("prec", [0, 1])
def test_largest_one_launch_block(sizes, prec):
    import paper_2306_00094_amd as dd
    print(f"case factor limit sizes={sizes} prec={prec}", flush=True)
    A, p = system(3, sizes, seed=2)
    s = dd.Solver(p, max_nrhs=1)
    s.factor(prec)
    for k, K in enumerate(p.kii):
        L = dd.dd_get_factor(s.ctx, prec, k, K.shape[0])
        ref = np.linalg.cholesky(K)
        assert np.abs(L - ref).max() <= (1e-12 if prec == dd.DD_FP64 else 2e-5) * np.abs(ref).max()
    b = np.random.default_rng(3).uniform(-1, 1, (1, p.n_dof))
    u = s.solve(torch.from_numpy(b).cuda(), prec=prec, opts=dd.dd_default_opts(tol=1e-13)).u.cpu().numpy()
    ref = np.linalg.solve(A, b[0])
    assert np.linalg.norm(u[0] - ref) <= (1e-10 if prec == dd.DD_FP64 else 1e-8) * np.linalg.norm(ref)
    s.close()
    j = max(sizes) - 7
    k = sizes.index(max(sizes))
    p.kii[k][j, j] = -1.0
    s = dd.Solver(p, max_nrhs=1)
    with pytest.raises(dd.DDError) as e:
        s.factor(prec)
    assert e.value.status == dd.DD_ENOTSPD and f"subdomain {k} not SPD at column {j}" in str(e.value)
    s.close()
