"""GPU test of the one-launch CG of small interfaces (dense Schur complement):
interface sizes around the multiples of 64 rows its workgroup is built from, and
around the last size it serves, against a dense FP64 solve and the stream
launches; columns in a batch equal to the same columns alone.  The systems have
condition numbers below 100 (diagonally dominant), so tolerance 1e-13 leaves a
relative error below 1e-10 (FP64) and 1e-8 (mixed)."""
import numpy as np
import pytest

from test_gpu_units import system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_gamma,sizes", [(1, (2, 3)), (63, (5, 1, 9)), (64, (70, 2)), (65, (16, 3, 40)),
                                           (192, (30, 4)), (193, (30, 4)), (384, (12, 3)), (385, (12, 3))])
@pytest.mark.parametrize("prec", [0, 1])
def test_small_interface(n_gamma, sizes, prec):
    import paper_2306_00094_amd as dd
    print(f"case direct n_gamma={n_gamma} prec={prec}", flush=True)
    A, p = system(n_gamma, sizes, seed=n_gamma)
    b = np.random.default_rng(2).uniform(-1, 1, (3, p.n_dof))
    b[1] = 0.0                                           # no iteration
    ref = np.linalg.solve(A, b.T).T
    bt = torch.from_numpy(b).to("cuda")
    s = dd.Solver(p, max_nrhs=3)
    s.factor(prec)
    opts = dd.dd_default_opts(tol=1e-13)
    r = s.solve(bt, prec=prec, opts=opts)
    u = r.u.cpu().numpy()
    k = s.solve(bt, prec=prec, opts=dd.dd_default_opts(tol=1e-13, launch=dd.DD_LAUNCH_KERNELS))
    gate = 1e-10 if prec == dd.DD_FP64 else 1e-8
    for j in (0, 2):
        assert np.linalg.norm(u[j] - ref[j]) <= gate * np.linalg.norm(ref[j])
        assert abs(r.info[j]["iters"] - k.info[j]["iters"]) <= (1 if prec == dd.DD_FP64 else 2)
        alone = s.solve(bt[j:j + 1].contiguous(), prec=prec, opts=opts)
        assert np.array_equal(alone.u.cpu().numpy()[0], u[j])
    assert np.all(u[1] == 0.0) and r.info[1]["iters"] == 0
    # a new factorisation forms S again; the iteration cap is kept
    s.factor(prec)
    assert np.array_equal(s.solve(bt, prec=prec, opts=opts).u.cpu().numpy(), u)
    if prec == dd.DD_FP64 and n_gamma > 60:
        c = s.solve(bt, opts=dd.dd_default_opts(tol=1e-13, max_it=2), raise_on_noconv=False)
        assert c.status == dd.DD_ENOCONV and [i["iters"] for i in c.info] == [2, 0, 2]
    s.close()
