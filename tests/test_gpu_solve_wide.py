"""Solves whose column slices end in a stage of fewer columns than a workgroup has
waves: blocks of 4160 rows (37 x 37 nodes, three responses), 32 slices of 130
columns.  Every wave of such a stage loads a column that exists
(tests/test_gemv_columns.py walks over all sizes); here the products' values: the
solution of Q_c x = r for r = Q_c x0, formed sparse on the CPU, must be x0 to the
condition number (3e4) times FP64 rounding of sums of 4160 terms."""
import numpy as np
import pytest

import workloads as W
from oracle import model as OM

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_06938_amd import dalia
    dalia.lib()
    return dalia


@pytest.mark.parametrize("two,nt", [(False, 2), (True, 4)])
def test_solve_with_a_short_last_stage(D, two, nt):
    wl = W.scaled("wide", 37, nt, 3, 1, 3000, seed=3)
    model = D.Model.from_workload(wl)
    assert model.bp == 4160
    perm = OM.bta_permutation(wl.nv, wl.ns, wl.nt, wl.nr)
    Q = OM.conditional_precision(wl, wl.theta)[perm][:, perm]
    x0 = np.random.default_rng(2).standard_normal((5, wl.N))
    r = (Q @ x0.T).T
    print(f"wide N={wl.N} two={two}", flush=True)
    ws = D.Workspace(model, two_sided=two)
    ws.assemble(wl.theta, D.DL_QC)
    _, info = ws.factor(D.DL_QC)
    R = torch.tensor(np.ascontiguousarray(r), device="cuda")
    x = ws.solve(R.clone(), refine_max=0)
    one = ws.solve(R[:1].clone(), refine_max=0)
    torch.cuda.synchronize()
    assert int(info[0]) == 0
    assert np.abs(x.cpu().numpy() - x0).max() <= 1e-9 * np.abs(x0).max()
    assert torch.equal(one[0], x[0])
