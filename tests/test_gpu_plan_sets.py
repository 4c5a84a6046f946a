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


@pytest.mark.parametrize("ksplit", [64, 256])
def test_forced_choices_reach_both_sets(D, ksplit):
    """Split products sum in another order, so a forced split shows in the bits: it
    must hold for the caller's blocks whether their set is built before or after,
    and for evaluations after a call made while that set is the active one."""
    wl = W.scaled("forced", 20, 4, 1, 2, 200, seed=4)  # bp = 448
    model = D.Model.from_workload(wl)

    def space():
        return D.Workspace(model, two_sided=True)

    plain = space()
    f_plain = plain.fobj(wl.theta)[1][:, :7].clone()
    own_plain = own_block(plain, wl, D)
    before, after = space(), space()
    before.force_split(ksplit)
    before.force_tile(128)
    own_block(after, wl, D)        # builds the second set, which is now active
    after.force_split(ksplit)
    after.force_tile(128)
    for ws in (before, after):
        assert ws.tile_counts()["tile64"] == 0 and ws.tile_counts()["tile128"] > 0
    f0, f1 = (ws.fobj(wl.theta)[1][:, :7].clone() for ws in (before, after))
    assert torch.equal(f0, f1) and not torch.equal(f0, f_plain)
    a, b = own_block(before, wl, D), own_block(after, wl, D)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert not torch.equal(a[1], own_plain[1])
    assert (a[1] - own_plain[1]).abs().max() <= 1e-10 * own_plain[1].abs().max()
    for ws in (before, after):
        assert ws.tile_counts()["tile64"] == 0  # also while the second set is active
    # and back
    for ws in (before, after):
        ws.force_split(0)
    for x, y in zip(own_block(before, wl, D), own_plain):
        assert torch.equal(x, y)
    assert torch.equal(after.fobj(wl.theta)[1][:, :7], f_plain)


@pytest.mark.parametrize("tile", [64, 128])
def test_only_the_lower_triangle_of_a_callers_diagonal_block_counts(D, tile):
    """A caller's symmetric diagonal blocks and tip, given in full, give the bits of
    their lower triangles, also where the products' tiles reach above a 64-wide
    diagonal tile."""
    wl = W.scaled("lower", 20, 3, 1, 2, 200, seed=6)
    model = D.Model.from_workload(wl)
    out = []
    for full in (False, True):
        ws = D.Workspace(model, selinv=True)
        ws.force_tile(tile)
        ws.assemble(wl.theta)
        for kind, t in ((0, 0), (0, 1), (0, 2), (3, 0)):
            A = torch.tril(ws.get_block(D.DL_QC, kind, t))
            ws.set_block(D.DL_QC, kind, t, A + torch.tril(A, -1).T if full else A)
        ld, info = ws.factor(D.DL_QC)
        assert int(info[0]) == 0
        out.append((ld.clone(), ws.solve().clone(), ws.selinv().clone()))
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("family,two", [("separable", False), ("diffusion", False),
                                        ("diffusion", True)])
def test_blocks_of_both_factors(D, family, two):
    """The blocks read back after a factorisation, of Q_c and of a kept Q_p: the
    inverse G_t of each diagonal block's factor and the coupling B_t G_t^T, against
    the blocks as they were assembled and a plain elimination in FP64."""
    wl = W.scaled("blocks", 10, 6, 1, 2, 100, seed=2, model=family)
    ws = D.Workspace(D.Model.from_workload(wl), keep_qp=True, two_sided=two)
    ws.assemble(wl.theta)
    mid = (wl.nt + 1) // 2 if two else wl.nt - 1
    want = {}
    for which in (D.DL_QP, D.DL_QC):
        Dt = [torch.tril(ws.get_block(which, 0, t)).cpu() for t in range(wl.nt)]
        Dt = [A + torch.tril(A, -1).T for A in Dt]
        Bt = [ws.get_block(which, 1, t).cpu() for t in range(wl.nt - 1)]
        order = [(t, t + 1, Bt[t]) for t in range(mid)]
        order += [(t, t - 1, Bt[t - 1].T) for t in range(wl.nt - 1, mid, -1)]
        for t, succ, B in order:
            G = torch.linalg.inv(torch.linalg.cholesky(Dt[t]))
            C = B @ G.T
            Dt[succ] = Dt[succ] - C @ C.T
            want[which, 0, t] = G
            if t < wl.nt - 1:  # (a last block's coupling is not a block of the caller's)
                want[which, 1, t] = C
        want[which, 0, mid] = torch.linalg.inv(torch.linalg.cholesky(Dt[mid]))
    ws.factor()
    for (which, kind, t), A in want.items():
        got = ws.get_block(which, kind, t).cpu()
        got = torch.tril(got) if kind == 0 else got
        assert (got - A).abs().max() <= 1e-11 * A.abs().max(), (which, kind, t)
