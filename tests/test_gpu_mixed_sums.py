"""f_obj of a separable univariate model with FP32 off-diagonal blocks.

log|Q_p| comes from one diagonal block without FP32 rounding, so all that FP32
does to log|Q_c| is in f.  The coupling products are summed in FP64 from the
exact stencil and rounded once (unbiased: their part of f grows with the square
root of the number of terms), the updates add their FP32 products in FP64 every
16 terms.  What is left is systematic: in each pivot D - sum c^2 the sum carries
the roundings of partial sums of at most 16 of its b terms, together less than
one FP32 rounding 2^-24 of the pivot.  Over the N pivots, f having half the
log-determinant: |f - f64| <= N 2^-24 / 2.  (FP32 chains over all b terms and a
stencil rounded to FP32 gave three times that.)"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_06938_amd import dalia
    dalia.lib()
    return dalia


# (nx, nt, nr, observations, two chains, Q_p kept, tile of all products)
CASES = [(5, 4, 0, 60, False, False, 0), (12, 10, 2, 800, False, False, 64),
         (20, 12, 2, 2400, True, False, 128), (20, 12, 2, 2400, True, True, 0),
         (30, 12, 3, 5000, True, False, 0)]


@pytest.mark.parametrize("nx,nt,nr,m,two,keep,tile", CASES)
def test_f_of_mixed_precision(D, nx, nt, nr, m, two, keep, tile):
    wl = W.scaled("mixsum", nx, nt, 1, nr, m, seed=3)
    model = D.Model.from_workload(wl)
    th = torch.tensor(wl.theta, device="cuda")
    ref = D.Workspace(model, two_sided=two).fobj(th)[1].cpu()[0]
    ws = D.Workspace(model, two_sided=two, mixed=True, keep_qp=keep)
    if tile:
        ws.force_tile(tile)
    f, parts, info = ws.fobj(th)
    assert int(info[0, 0]) == 0
    got = parts.cpu()[0]
    bound = 0.5 * wl.N * 2.0 ** -24
    print(nx, "f", float(got[0] - ref[0]), "bound", bound)
    assert abs(float(got[0] - ref[0])) <= bound
    assert abs(float(got[1] - ref[1])) <= 1e-11 * abs(float(ref[1]))


def test_couplings_keep_their_own_theta(D):
    """Q_p assembled for another theta between Q_c's assembly and factor."""
    wl = W.scaled("mixsum", 13, 5, 1, 2, 200, seed=3)
    model = D.Model.from_workload(wl)
    th = np.asarray(wl.theta)
    lds = []
    for other in (False, True):
        ws = D.Workspace(model, mixed=True)
        ws.assemble(th, D.DL_QC)
        if other:
            ws.assemble(th + 0.3, D.DL_QP)
        ld, info = ws.factor(D.DL_QC)
        assert int(info[-1]) == 0
        lds.append(float(ld[-1]))
    assert lds[0] == lds[1]


def test_batch_of_models_with_and_without_fp64_sums(D):
    """One and three responses in one launch: each as if alone."""
    wls = [W.scaled("m1", 14, 4, 1, 2, 150, seed=1), W.scaled("m3", 8, 4, 3, 1, 60, seed=2)]
    models = [D.Model.from_workload(w) for w in wls]
    th = [torch.tensor(w.theta, device="cuda") for w in wls]
    alone = [D.Workspace(m, mixed=True).fobj(t)[1].cpu()[0] for m, t in zip(models, th)]
    both = D.Workspace(models, mixed=True).fobj(torch.cat(th))[1].cpu()
    for k in range(2):
        assert torch.equal(both[k], alone[k])
