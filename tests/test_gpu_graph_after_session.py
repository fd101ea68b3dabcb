"""GPU test of graph-replayed solves around a batch session on one context.  A
captured CG graph holds the addresses of the work vectors; a session exchanges
them (column layouts, direction buffers).  The solve after the session gives the
bits, iterations and refinement steps of the one before it."""
import numpy as np
import pytest

from test_gpu_units import system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def session(dd, s, b, prec, opts, slots, iters):
    """Slots admitted one after the other, iters iterations after each, and closed
    with them running."""
    dd.dd_batch_begin(s.ctx, prec, opts)
    for sl in slots:
        dd.dd_batch_admit(s.ctx, [sl], b[sl:sl + 1], b.shape[1])
        dd.dd_batch_step(s.ctx, iters, 8)
    dd.dd_batch_end(s.ctx)


@pytest.mark.parametrize("tiles", [0, 1])
@pytest.mark.parametrize("prec,slots,iters", [(0, (0,), 1), (0, (0, 1, 3, 7), 2), (1, (0, 1, 3, 7), 2)])
def test_graph_solve_after_session(prec, slots, iters, tiles):
    import paper_2306_00094_amd as dd
    print(f"case graph after session prec={prec} slots={slots} iters={iters} tiles={tiles}", flush=True)
    A, p = system(100, (7, 20, 31), seed=9)
    b = torch.from_numpy(np.random.default_rng(10).uniform(-1, 1, (8, len(A)))).cuda()
    s = dd.Solver(p, max_nrhs=8)
    s.factor(dd.DD_FP64)
    if prec == dd.DD_MIXED:
        s.factor(prec)
    opts = dd.dd_default_opts(tol=1e-13, launch=dd.DD_LAUNCH_GRAPH, tiles=tiles, reliable=0)
    before = s.solve(b, prec=prec, opts=opts)
    assert all(i["converged"] and not i["used_fallback"] for i in before.info)
    assert prec == dd.DD_FP64 or min(i["refine_steps"] for i in before.info) >= 2
    u = before.u.cpu().numpy()
    session(dd, s, b, prec, dd.dd_default_opts(tol=1e-12), slots, iters)
    after = s.solve(b, prec=prec, opts=opts, raise_on_noconv=False)
    assert after.status == dd.DD_OK
    assert after.info == before.info
    assert np.array_equal(after.u.cpu().numpy(), u)
    s.close()
