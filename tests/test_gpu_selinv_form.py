"""Selected inversion of large univariate blocks, whose steps multiply triangles
(X = G^T (I + [C; R]^T X [C; R]) G): the smallest padded block sizes that take
this form with one chain (38 x 38 nodes) and with two (33 x 33) and the general form
below them, with and without arrow rows, one time step, and a caller's dense
sub-diagonal block, all against a dense inverse.  The tolerance allows for cond(Q) eps (about 1e5 here)."""
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


@pytest.mark.parametrize("nx,nt,nr,two,dense", [(36, 3, 2, False, False), (36, 4, 0, True, False),
                                                (37, 4, 1, True, False), (36, 1, 1, False, False),
                                                (36, 1, 0, False, False), (36, 2, 1, False, True),
                                                (38, 3, 2, False, False), (38, 1, 0, False, False),
                                                (38, 2, 1, False, True), (33, 4, 0, True, False),
                                                (32, 4, 2, True, False), (33, 4, 1, True, True)])
def test_variances_of_large_blocks(D, nx, nt, nr, two, dense):
    wl = W.scaled("selform", nx, nt, 1, nr, 700, seed=13)
    ref = OF.fobj_parts(wl, wl.theta, return_factors=True)
    perm = OM.bta_permutation(wl.nv, wl.ns, wl.nt, wl.nr)
    Q = torch.tensor(ref["Qc"].toarray()[np.ix_(perm, perm)])
    model = D.Model.from_workload(wl)
    ws = D.Workspace(model, selinv=True, two_sided=two)
    ws.assemble(wl.theta)
    if dense:
        b = wl.b
        g = torch.Generator().manual_seed(1)
        E = 1e-3 * torch.diagonal(Q).min() * torch.randn(b, b, generator=g, dtype=torch.float64)
        Q[b:2 * b, :b] += E
        Q[:b, b:2 * b] = Q[b:2 * b, :b].T
        ws.set_block(D.DL_QC, 1, 0, Q[b:2 * b, :b].contiguous().cuda())
    _, info = ws.factor(D.DL_QC)
    var = ws.selinv().cpu()
    assert int(info[0]) == 0
    want = torch.diagonal(torch.linalg.inv(Q))
    assert ((var - want).abs() <= 1e-9 * want).all()
    if not dense:
        again = D.Workspace([model, model], selinv=True, two_sided=two)
        again.assemble(np.concatenate([wl.theta, wl.theta]))
        again.factor()
        v2 = again.selinv().cpu()
        assert torch.equal(v2[:wl.N], var) and torch.equal(v2[wl.N:], var)


@pytest.mark.parametrize("nx,nt,two", [(38, 2, False), (33, 4, True)])
def test_forced_tiles_and_splits_of_the_triangles_products(D, nx, nt, two):
    """Tiles of 128 reach above the 64-wide diagonal tiles, and split pieces are cut
    without regard to the rows that begin late: the same bits for either tile, and
    the unsplit variances to the rounding of sums in pieces."""
    wl = W.scaled("selforce", nx, nt, 1, 2, 500, seed=3)
    model = D.Model.from_workload(wl)
    var = {}
    for tile in (64, 128):
        for ksplit in (0, 256):
            ws = D.Workspace(model, selinv=True, two_sided=two)
            ws.force_tile(tile)
            ws.force_split(ksplit)
            ws.assemble(wl.theta)
            ws.factor()
            var[tile, ksplit] = ws.selinv().cpu()
    for ksplit in (0, 256):
        assert torch.equal(var[64, ksplit], var[128, ksplit])
    np.testing.assert_allclose(var[64, 256], var[64, 0], rtol=1e-11)
