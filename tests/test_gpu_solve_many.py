"""Several right-hand sides per pass over the factor.

bta_solve takes up to four caller vectors at once when no refinement is asked
for.  A vector's result must not depend on how many share its pass, on how
they fall into groups, or on the matrices of a batch: every count from 1 to 9
is compared bit for bit with one vector at a time, and with a dense solve.
The block sizes cover an odd and an even number of 64-wide tiles (a row block
of the matrix-vector products is two tiles), the tip none and one, one time
step, and both chains.
"""
import numpy as np
import pytest

import workloads as W
from oracle import fobj as OF
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


def dense(wl):
    ref = OF.fobj_parts(wl, wl.theta, return_factors=True)
    perm = OM.bta_permutation(wl.nv, wl.ns, wl.nt, wl.nr)
    return ref["Qc"].toarray()[np.ix_(perm, perm)]


# (name, nx, nt, nv, nr, observations, two chains, mixed)
SHAPES = [("one_tile", 6, 4, 1, 2, 50, True, False),
          ("three_tiles_chain", 12, 3, 1, 1, 90, False, False),
          ("four_tiles_no_tip", 9, 3, 3, 0, 80, True, False),
          ("one_step", 7, 1, 3, 2, 60, True, False),
          ("mixed", 10, 5, 2, 1, 90, True, True)]


@pytest.mark.parametrize("name,nx,nt,nv,nr,m,two,mixed", SHAPES, ids=[s[0] for s in SHAPES])
def test_grouped_vectors_equal_single_ones(D, name, nx, nt, nv, nr, m, two, mixed):
    wl = W.scaled("many_" + name, nx, nt, nv, nr, m, seed=17)
    ws = D.Workspace(D.Model.from_workload(wl), mixed=mixed, two_sided=two)
    ws.assemble(wl.theta)
    ws.factor()
    rng = np.random.default_rng(3)
    R = torch.tensor(rng.standard_normal((9, wl.N)), device="cuda")
    one = torch.stack([ws.solve(R[i].clone(), refine_max=0) for i in range(9)])
    if not mixed:  # the factor of the mixed mode is 32-bit
        want = np.linalg.solve(dense(wl), R.cpu().numpy().T).T
        np.testing.assert_allclose(one.cpu().numpy(), want, rtol=0,
                                   atol=1e-9 * np.abs(want).max())
    for n in range(1, 10):
        got = ws.solve(R[:n].clone(), refine_max=0)
        assert torch.equal(got, one[:n]), n
        # the workspace holds the last solution
        assert torch.equal(ws.mean(), one[n - 1]), n


def test_grouped_vectors_in_a_batch(D):
    wls = [W.scaled("many_batch%d" % i, nx, nt, 1, nr, 50, seed=5 + i)
           for i, (nx, nt, nr) in enumerate([(6, 4, 2), (12, 3, 1), (9, 1, 0)])]
    ws = D.Workspace([D.Model.from_workload(w) for w in wls])
    theta = np.concatenate([np.asarray(w.theta, dtype=np.float64).ravel() for w in wls])
    ws.assemble(theta)
    ws.factor()
    rng = np.random.default_rng(4)
    R = torch.tensor(rng.standard_normal((6, ws.N_total)), device="cuda")
    one = torch.stack([ws.solve(R[i].clone()) for i in range(6)])
    assert torch.equal(ws.solve(R.clone()), one)
    off = 0
    for w in wls:
        r = R[:, off:off + w.N].cpu().numpy()
        x = one[:, off:off + w.N].cpu().numpy()
        want = np.linalg.solve(dense(w), r.T).T
        np.testing.assert_allclose(x, want, rtol=0, atol=1e-9 * np.abs(want).max())
        off += w.N
