"""GPU tests of the three-launch CG iteration on small systems, which run the
one-launch CG unless a launch mode is asked for: stream launches and graph replays
of it against the CPU FP64 oracle, FP64 error <= 1e-10 and mixed <= 1e-8 relative
to the monolithic solution; iteration counts within 2 of the oracle's; a column's
bits the same alone and in batches of 3 and of 64; zero and repeated columns."""
import functools

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SYSTEMS = {
    "1d-4strips": lambda: workloads.spec_1d(n=256, strips=4, nrhs=64),
    "1d-ragged": lambda: workloads.spec_1d(n=100, delta=0.07, strips=3, nrhs=64),
    "2d-const": lambda: workloads.spec_2d_const(n=32, cuts=(2, 2), nrhs=64, seed_base=7000),
    "2d-frac": lambda: workloads.spec_2d_frac(n=32, cuts=(2, 2), nrhs=64),
}


@functools.lru_cache(maxsize=None)
def problem(name):
    spec = SYSTEMS[name]()
    wl = workloads.build(spec)
    b = workloads.rhs(spec)
    return wl, b, oracle.monolithic_solve(wl.asm.A, b)


def dev(b):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(b).T)).to("cuda:0").contiguous()


@pytest.mark.parametrize("name", list(SYSTEMS))
@pytest.mark.parametrize("launch", [1, 3])
@pytest.mark.parametrize("prec", [0, 1])
def test_three_launch_iteration(name, launch, prec):
    import paper_2306_00094_amd as dd
    wl, b, uref = problem(name)
    print(f"case stream launches {name} launch={launch} prec={prec}", flush=True)
    assert wl.dd.n_gamma <= 384
    s = dd.Solver(wl.dd, max_nrhs=64)
    s.factor(prec)
    opts = dd.dd_default_opts(tol=1e-13, launch=launch)
    r = s.solve(dev(b), prec=prec, opts=opts)
    u = r.u.cpu().numpy()
    assert oracle.rel_err(u.T, uref).max() <= (1e-10 if prec == dd.DD_FP64 else 1e-8)
    if prec == dd.DD_FP64:
        _, its, _ = oracle.DDOracle(wl.dd).solve(b[:, :4], tol=1e-13)
        assert all(abs(r.info[j]["iters"] - int(its[j])) <= 2 for j in range(4)), (r.info[:4], its)
    for cols in ([37], [0, 37, 63]):
        alone = s.solve(dev(b[:, cols]), prec=prec, opts=opts).u.cpu().numpy()
        assert np.array_equal(alone, u[cols]), cols
    z = np.zeros((b.shape[0], 3))
    z[:, 1] = z[:, 2] = b[:, 5]
    r = s.solve(dev(z), prec=prec, opts=opts)
    v = r.u.cpu().numpy()
    assert np.all(v[0] == 0.0) and r.info[0]["iters"] == 0
    assert np.array_equal(v[1], u[5]) and np.array_equal(v[2], u[5])
    s.close()
