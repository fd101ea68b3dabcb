"""GPU test of the FETI iteration at column counts around its groups of 8 columns
(the deflation by 8 columns and 64 rows, the dots by column), with floating
subdomains of one (constant kernel) and three (peridynamics) rigid motions."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_feti import dev, problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["1d", "2d-const", "2d-pd"])
def test_feti_column_counts(name):
    """Error <= 1e-10 against the monolithic solution at tolerance 1e-12, a zero
    load gives zero without an iteration, and max_it ends the loop unconverged."""
    import paper_2306_00094_amd as dd
    spec, wl, fp, b, uref = problem(name)
    s = dd.FetiSolver(wl.dd, fp, max_nrhs=64)
    s.factor()
    for m in (1, 7, 8, 9, 17, 64):
        print(f"case feti widths {name} columns={m}", flush=True)
        scale = 1.0 + np.arange(m)
        scale[m // 2] = 0.0 if m > 1 else 1.0
        cols = np.arange(m) % b.shape[1]
        r = s.solve(dev(b[:, cols] * scale), tol=1e-12, max_it=500)
        u = r.u.cpu().numpy().T
        ref = uref[:, cols] * scale
        nz = scale > 0
        assert oracle.rel_err(u[:, nz], ref[:, nz]).max() <= 1e-10
        assert not u[:, ~nz].any() and all(r.info[j]["iters"] == 0 for j in np.nonzero(~nz)[0])
        assert all(i["converged"] for i in r.info)
    with pytest.raises(dd.DDError) as ei:
        s.solve(dev(b[:, :1]), tol=1e-12, max_it=2)
    assert ei.value.status == dd.DD_ENOCONV
    s.close()
