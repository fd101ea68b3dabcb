"""GPU test of solves of different schedules one after the other on one context: the
count of p^T q sums that the last interface-row launch of one left must not reach the
first launch of the next (up to 640 block sums of the tiled rows, where the
three-launch iteration reads group sums).  Each solve gives the bits of the same
solve on a context of its own."""
import numpy as np
import pytest

from test_gpu_tiled_sizes import system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_gamma", [400, 10240, 10241])
@pytest.mark.parametrize("prec", [0, 1])
def test_schedules_in_turn(n_gamma, prec):
    import paper_2306_00094_amd as dd
    _, p = system(n_gamma, (40, 17, 33))
    b = torch.from_numpy(np.random.default_rng(1).uniform(-1, 1, (64, p.n_dof))).cuda()

    def solve(s, m, **o):
        print(f"case schedules in turn n_gamma={n_gamma} prec={prec} columns={m} {o}", flush=True)
        return s.solve(b[:m].contiguous(), prec=prec, opts=dd.dd_default_opts(tol=1e-10, **o)).u.cpu().numpy()

    def context():
        s = dd.Solver(p, max_nrhs=64)
        s.factor(prec)
        return s

    turns = [(64, dict(tiles=1)), (64, dict(tiles=0)), (8, dict(tiles=1, launch=dd.DD_LAUNCH_GRAPH)),
             (1, dict()), (8, dict(tiles=1)), (64, dict(tiles=0, launch=dd.DD_LAUNCH_GRAPH)), (3, dict())]
    s = context()
    for m, o in turns:
        u = solve(s, m, **o)
        alone = context()
        assert np.array_equal(solve(alone, m, **o), u), (m, o)
        alone.close()
    s.close()
