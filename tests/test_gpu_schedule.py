"""GPU tests of which schedule a solve of a small interface runs (the phase timing
tells them apart: the one-launch CG is one DD_PHASE_LOOP and no interface-row
launch) and of the autotuner's report of it."""
import numpy as np
import pytest

from test_gpu_units import system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def one_launch(dd, s, b, prec, opts):
    """(whether the CG ran in one launch, the solution)"""
    dd.dd_set_timing(s.ctx, 31)
    u = s.solve(b, prec=prec, opts=opts).u.cpu().numpy()
    n = dd.dd_get_timing(s.ctx)[1]
    dd.dd_set_timing(s.ctx, 0)
    assert (n[dd.DD_PHASE_LOOP] > 0) != (n[dd.DD_PHASE_GAMMA] > 0), n
    return n[dd.DD_PHASE_LOOP] > 0, u


@pytest.mark.parametrize("prec", [0, 1])
def test_sizes_served_in_one_launch(prec):
    """Up to 384 interface rows by default, never when a launch mode is asked for."""
    import paper_2306_00094_amd as dd
    for n_gamma in (1, 384, 385):
        print(f"case schedule n_gamma={n_gamma} prec={prec}", flush=True)
        _, p = system(n_gamma, (12, 3), seed=1)
        s = dd.Solver(p, max_nrhs=1)
        s.factor(prec)
        b = torch.from_numpy(np.random.default_rng(2).uniform(-1, 1, (1, p.n_dof))).cuda()
        assert one_launch(dd, s, b, prec, dd.dd_default_opts(tol=1e-10))[0] == (n_gamma <= 384)
        assert not one_launch(dd, s, b, prec, dd.dd_default_opts(tol=1e-10, launch=dd.DD_LAUNCH_KERNELS))[0]
        s.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_reported_schedule_given_back(prec):
    """apply and launch as the autotuner reports them, given to a solve on another
    context, run the schedule it chose: the same bits and launches."""
    import paper_2306_00094_amd as dd
    print(f"case tuned schedule given back prec={prec}", flush=True)
    _, p = system(100, (70, 3, 40), seed=1)
    b = torch.from_numpy(np.random.default_rng(2).uniform(-1, 1, (1, p.n_dof))).cuda()
    s, t = dd.Solver(p, max_nrhs=1), dd.Solver(p, max_nrhs=1)
    for x in (s, t):
        x.factor(prec)
    r = s.autotune(prec)
    want = one_launch(dd, s, b, prec, dd.dd_default_opts(tol=1e-10))
    assert want[0] and r["launch"] == dd.DD_LAUNCH_AUTO and r["three_launch"] == 0
    itol = r["inner_tol"] if prec == dd.DD_MIXED else 0.0
    got = one_launch(dd, t, b, prec, dd.dd_default_opts(tol=1e-10, apply=r["apply"], launch=r["launch"],
                                                        inner_tol=itol))
    assert got[0] and np.array_equal(got[1], want[1])
    s.close()
    t.close()
