"""GPU tests of batch sessions: a session after one whose iterate became NaN, and
sessions on contexts with units (max_nrhs >= 8) at block
edges and column counts on both sides of each layout width."""
import numpy as np
import pytest

from test_gpu_units import system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dd():
    import paper_2306_00094_amd as dd
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dd.load_library()
    return dd


def session(dd, s, b, prec, opts, width):
    """All columns of b ([column][row], on the device) through one session."""
    m, n = b.shape
    u = torch.empty_like(b)
    dd.dd_batch_begin(s.ctx, prec, opts)
    dd.dd_batch_admit(s.ctx, list(range(m)), b, n)
    for _ in range(500):
        if dd.DD_SLOT_RUNNING not in dd.dd_batch_step(s.ctx, 4, width)[:m]:
            break
    info = dd.dd_batch_retire(s.ctx, list(range(m)), u, n)
    dd.dd_batch_end(s.ctx)
    return u.cpu().numpy(), info


@pytest.mark.parametrize("prec", [0, 1])
def test_session_after_nan(prec):
    """A load of NaN leaves a NaN iterate in its slot; the next session in that
    slot gives the bits of a session on a fresh context."""
    dd = _dd()
    A, p = system(17, (33, 16, 1), seed=5)
    b = torch.from_numpy(np.random.default_rng(6).uniform(-1, 1, (1, len(A)))).cuda()
    opts = dd.dd_default_opts(tol=1e-13, fp64_fallback=0)
    out = []
    for first in (b, torch.full_like(b, float("nan"))):
        s = dd.Solver(p, max_nrhs=1)
        s.factor(prec)
        print(f"case session after NaN prec={prec}", flush=True)
        session(dd, s, first, prec, opts, 1)
        out.append(session(dd, s, b, prec, opts, 1)[0])
        s.close()
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("n_gamma,sizes", [(1, (1, 2)), (16, (5, 1)), (17, (33, 16, 1)), (100, (7, 20, 31))])
@pytest.mark.parametrize("prec,gather32", [(0, -1), (1, 0), (1, 1)])
def test_sessions_on_units(n_gamma, sizes, prec, gather32):
    """1 to 33 columns of a session: the solution of systems with condition
    numbers below 100 (tolerance 1e-13: error below 1e-10 in FP64 and 1e-8 in
    mixed precision with a wide margin), and a column's bits independent of the
    others."""
    dd = _dd()
    A, p = system(n_gamma, sizes, seed=7)
    s = dd.Solver(p, max_nrhs=64)
    s.factor(prec)
    opts = dd.dd_default_opts(tol=1e-13, gather32=gather32)
    b = np.random.default_rng(8).uniform(-1, 1, (33, len(A)))
    ref = np.linalg.solve(A, b.T).T
    one = None
    for m in (1, 2, 7, 9, 16, 17, 33):
        print(f"case session on units n_gamma={n_gamma} prec={prec} gather32={gather32} columns={m}", flush=True)
        u, info = session(dd, s, torch.from_numpy(b[:m].copy()).cuda(), prec, opts, 64)
        assert all(i["converged"] for i in info)
        err = np.linalg.norm(u - ref[:m], axis=1) / np.linalg.norm(ref[:m], axis=1)
        assert err.max() <= (1e-8 if prec else 1e-10), err
        one = u[0] if one is None else one
        assert np.array_equal(u[0], one)
    s.close()
