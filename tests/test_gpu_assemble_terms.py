"""Assembly where its waves' cases meet: no observation at all, several rows on one
node (more than one pass of 32), a row whose nodes are far apart (outside the
stencil, where an entry is not one of the wave's own), the same node twice in
one row, three responses with covariates, and the diffusion stencil (two
entries a lane).  Every block is compared with the oracle's matrix, to rounding."""
import dataclasses

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


@pytest.mark.parametrize("nv,nr,model", [(1, 0, "separable"), (1, 2, "separable"),
                                         (3, 3, "separable"), (3, 1, "diffusion"),
                                         (2, 0, "diffusion")])
def test_blocks_of_odd_observations(D, nv, nr, model):
    nx, nt = 9, 3
    wl = W.scaled("terms", nx, nt, nv, nr, 60, seed=3, model=model)
    rng = np.random.default_rng(0)
    out = []
    for j, r in enumerate(wl.responses):
        nodes = np.array(r.nodes, copy=True)
        t = np.array(r.t, copy=True)
        n = nodes.shape[0]
        if j == 0:
            nodes[:45] = nodes[0]  # 45 rows on the same three nodes
            t[:45] = 1
            nodes[45] = (0, nx * nx - 1, 40)  # far apart
            nodes[46] = (7, 7, 8)  # one node twice
            t[47:] = np.where(t[47:] == 2, 0, t[47:])  # a step without observations
        out.append(dataclasses.replace(r, nodes=nodes, t=t))
    wl = dataclasses.replace(wl, responses=out)
    ref = OF.fobj_parts(wl, wl.theta, return_factors=True)
    perm = OM.bta_permutation(wl.nv, wl.ns, wl.nt, wl.nr)
    Q = ref["Qc"].toarray()[np.ix_(perm, perm)]
    ws = D.Workspace(D.Model.from_workload(wl), keep_qp=True)
    ws.assemble(wl.theta)
    b = wl.b
    tol = 1e-12 * np.abs(Q).max()
    for t in range(nt):
        got = ws.get_block(D.DL_QC, 0, t).cpu().numpy()
        np.testing.assert_allclose(np.tril(got), np.tril(Q[t * b:(t + 1) * b, t * b:(t + 1) * b]),
                                   rtol=0, atol=tol)
        assert np.all(np.triu(got, 1) == 0)
        if t + 1 < nt:
            np.testing.assert_allclose(ws.get_block(D.DL_QC, 1, t).cpu().numpy(),
                                       Q[(t + 1) * b:(t + 2) * b, t * b:(t + 1) * b], rtol=0,
                                       atol=tol)
        if nr:
            np.testing.assert_allclose(ws.get_block(D.DL_QC, 2, t).cpu().numpy(),
                                       Q[nt * b:, t * b:(t + 1) * b], rtol=0, atol=tol)
    # an evaluation, which leaves the zeros of the sub-diagonal blocks unwritten
    f = D.Workspace(D.Model.from_workload(wl)).fobj(wl.theta)[0]
    want = OF.fobj_parts(wl, wl.theta)["f"]
    assert abs(float(f.cpu().ravel()[0]) - want) <= 1e-9 * abs(want)
