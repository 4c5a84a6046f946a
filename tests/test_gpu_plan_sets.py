"""A workspace's two plan sets: the one of assembled sub-diagonal blocks, which
evaluations and captured graphs use, and the one of a caller's own (set_block)
blocks, built at the first such call."""
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


def own_block(ws, wl, D):
    """Factor and solve with a sub-diagonal block set to the value it has."""
    ws.assemble(wl.theta)
    ws.set_block(D.DL_QC, 1, 0, ws.get_block(D.DL_QC, 1, 0).clone())
    ld, info = ws.factor(D.DL_QC)
    assert int(info[0]) == 0
    return ld.clone(), ws.solve().clone()


@pytest.mark.parametrize("nx,nt,two", [(24, 3, False), (26, 5, True)])  # bp = 576, 704
def test_split_graph_replays_after_a_callers_block(D, nx, nt, two):
    """The split products' partial tiles are sized per plan set, and a captured
    graph keeps the address of its own: the set of the caller's blocks, which
    needs more of them, is built between two replays."""
    wl = W.scaled("plan_sets", nx, nt, 1, 2, 200, seed=8)
    model = D.Model.from_workload(wl)
    theta = W.random_theta_near(wl.theta, 0.1, seed=2)
    ref = D.Workspace(model, splitk=True, two_sided=two)
    want = [ref.fobj(t)[1].clone() for t in (wl.theta, theta)]
    ws = D.Workspace(model, graph=True, splitk=True, two_sided=two)
    f0 = ws.fobj(wl.theta)[1].clone()
    assert torch.equal(f0[:, :7], want[0][:, :7])
    own = own_block(ws, wl, D)
    keep = torch.full((1 << 21,), 7.0, device="cuda", dtype=torch.float64)
    for rep in range(3):
        for t, w in zip((wl.theta, theta), want):
            assert torch.equal(ws.fobj(t)[1][:, :7], w[:, :7]), rep
        again = own_block(ws, wl, D)
        assert all(torch.equal(a, b) for a, b in zip(own, again)), rep
    assert (keep == 7.0).all()
