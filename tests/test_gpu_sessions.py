"""GPU test of batch sessions: a session after one whose iterate became NaN."""
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
