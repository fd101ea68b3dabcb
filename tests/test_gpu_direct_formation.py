"""GPU test of how the dense Schur complement of a small interface is formed (by
the first solve after a factorisation): interface rows with more entries than a
workgroup has threads, interface columns in several subdomains, K_GG with and
without repeated entries, against a dense FP64 solve (condition numbers below 100:
tolerance 1e-13 leaves a relative error below 1e-10 in FP64 and 1e-8 in mixed
precision); and what it costs beside a solve."""
import time

import numpy as np
import pytest

from test_gpu_units import system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_gamma,sizes", [(40, (900, 3, 700)), (64, (17, 1, 300, 16)), (300, (33, 2, 500, 48))])
@pytest.mark.parametrize("repeats", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
def test_formation(n_gamma, sizes, repeats, prec):
    import paper_2306_00094_amd as dd
    print(f"case formation n_gamma={n_gamma} sizes={sizes} repeats={repeats} prec={prec}", flush=True)
    A, p = system(n_gamma, sizes, seed=3)
    if not repeats:
        p.kgg = p.kgg.copy()
        p.kgg.sum_duplicates()
    b = np.random.default_rng(4).uniform(-1, 1, (2, p.n_dof))
    ref = np.linalg.solve(A, b.T).T
    s = dd.Solver(p, max_nrhs=2)
    s.factor(prec)
    u = s.solve(torch.from_numpy(b).cuda(), prec=prec, opts=dd.dd_default_opts(tol=1e-13)).u.cpu().numpy()
    err = np.linalg.norm(u - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= (1e-10 if prec == dd.DD_FP64 else 1e-8), err
    s.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_first_solve_costs_little_more(prec):
    """60 interface rows with 1 150 entries each: the first solve after a
    factorisation takes at most three times a later one (about twice; 7 times with
    one workgroup per row going through its entries one by one)."""
    import paper_2306_00094_amd as dd
    print(f"case first solve prec={prec}", flush=True)
    _, p = system(60, (960, 1, 960, 960), seed=3)
    s = dd.Solver(p, max_nrhs=1)
    b = torch.from_numpy(np.random.default_rng(4).uniform(-1, 1, (1, p.n_dof))).cuda()
    u = torch.empty_like(b)
    t = [[], []]
    for _ in range(8):
        s.factor(prec)
        for k in range(2):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            s.solve(b, prec=prec, u=u)
            torch.cuda.synchronize()
            t[k].append(time.perf_counter() - t0)
    first, later = min(t[0]), min(t[1])
    print(f"first {first * 1e6:.0f} us, later {later * 1e6:.0f} us", flush=True)
    assert first <= 3.0 * later
    s.close()
