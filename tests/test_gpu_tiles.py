"""Element kernels at the edges of their tiles: one element, one short of a workgroup's
elements, exactly full, one over, and several workgroups with a ragged last one."""
import numpy as np
import pytest

from _support import LAM, MU, ensure_built, gpu_available, inputs, print_case, rel, t2n

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

TOL = {"f64": 1e-12, "f32": 1e-5}  # those of the operator tests
# elements a transfer workgroup takes: 2 x (9, 1, 2) for fine orders 2..4
SIZES = [(1, 1, 1), (3, 1, 1), (4, 1, 1), (5, 1, 1), (7, 1, 1), (17, 1, 1), (2, 3, 3), (19, 1, 1), (5, 3, 2)]


def _hierarchy(n, orders, **kw):
    from paper_2204_01722_amd.problem import Hierarchy
    ensure_built()
    m = inputs.box_mesh(n, orders[0], jitter=0.05, seed=2204)
    return m, Hierarchy(m, list(orders), faces={"x0": (1, 0, 1)}, **kw)


@pytest.mark.parametrize("orders", [(2, 1), (3, 1), (4, 2), (4, 3), (3, 2), (4, 1)])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_transfers_at_tile_edges(orders, precision):
    """Prolongation and restriction against the oracle's interpolation matrix."""
    import torch
    from oracle import mg as omg
    from paper_2204_01722_amd.binding import hpmg_prolong_add, hpmg_restrict
    dt = torch.float64 if precision == "f64" else torch.float32
    for n in SIZES:
        print_case("transfer_tiles", n=n, orders=orders, precision=precision)
        m, H = _hierarchy(n, orders)
        f, c = H.ops
        Pm = omg.prolongation(H.topos[0], orders[0] + 1, f.n_nodes, H.topos[1], orders[1] + 1, c.n_nodes)
        mf, mc = 1.0 - H.masks[0].reshape(-1), 1.0 - H.masks[1].reshape(-1)
        x, y, r = (inputs.random_vector(k, s) for k, s in ((c.n_nodes, 1), (f.n_nodes, 2), (f.n_nodes, 3)))
        dev = lambda v: torch.from_numpy(v).to("cuda", dt)  # noqa: E731
        got = t2n(hpmg_prolong_add(c, f, dev(x), dev(y), precision))
        assert rel(got, y.reshape(-1) + mf * (Pm @ (mc * x.reshape(-1)))) < TOL[precision]
        got = t2n(hpmg_restrict(f, c, dev(r), precision))
        assert rel(got, mc * (Pm.T @ (mf * r.reshape(-1)))) < TOL[precision]


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("mode", ["stored", "recompute"])
def test_diagonal_and_adjoint_at_tile_edges(p, mode):
    """Diagonal, and the adjoint with its per-element parameter gradients, in both
    precisions against the oracle."""
    import torch
    from oracle import fem
    for n in [(1, 1, 1), (3, 1, 1), (5, 1, 1), (10, 1, 1), (11, 3, 1)]:
        print_case("diagonal_adjoint_tiles", n=n, p=p, mode=mode)
        E = int(np.prod(n))
        mu_e, lam_e = inputs.loguniform_materials(E, seed=4)
        m, H = _hierarchy(n, (p,), mu_e=mu_e, lam_e=lam_e)
        op = H.fine
        u, w = inputs.config1_u(m, amplitude=0.05), inputs.random_vector(m.n_nodes, 5)
        ut, wt = torch.from_numpy(u).cuda(), torch.from_numpy(w).cuda()
        op.residual(ut, store_state=True)
        op.state_cast_f32()
        d = fem.make_disc(m.coords, m.elem_nodes, p + 1)
        diag = fem.diagonal(d, u, mu_e, lam_e, H.masks[0])
        ref = fem.residual_vjp(d, u, w, mu_e, lam_e, H.masks[0])
        for prec in ("f64", "f32"):
            assert rel(t2n(op.diagonal(prec)), diag) < TOL[prec]
            ww = wt if prec == "f64" else wt.float()
            got = op.residual_vjp(ut, ww, mode=mode, precision=prec)
            for g, r in zip(got, ref):
                assert rel(t2n(g), r) < TOL[prec]
            alone = op.residual_vjp(ut, ww, mode=mode, precision=prec, want_params=False)
            assert alone[1] is None and torch.equal(alone[0], got[0])


@pytest.mark.parametrize("p, n", [(4, (24, 25, 25)), (4, (25, 25, 25)), (2, (43, 43, 43)), (3, (32, 32, 31))])
def test_state_on_both_sides_of_the_cache(p, n):
    """A residual whose state stays in the last-level cache or streams past it (more than
    240 MiB): the residual of the form without a state bit for bit, and a stored linearisation
    that acts as the recomputed one, also in a ragged last tile."""
    import torch
    print_case("state_stream", n=n, p=p)
    m, H = _hierarchy(n, (p,))
    op = H.fine
    u, du = (torch.from_numpy(v).cuda() for v in (inputs.config1_u(m, amplitude=0.05),
                                                  inputs.random_vector(m.n_nodes, 5)))
    r = op.residual(u, store_state=True)
    assert torch.equal(r, op.residual(u, store_state=False))
    assert rel(t2n(op.jacobian(du)), t2n(op.jacobian(du, mode="recompute", u=u))) < TOL["f64"]
    assert op.query_flags() == 0


@pytest.mark.parametrize("n", [17, 25])
def test_vcycle_state_kept_in_cache(n):
    """V-cycles that load the linearisation so that it stays in the cache (48 to 168 MiB: FP64
    on 17^3, FP32 on 25^3) against the other precision, whose size takes the other loads."""
    import torch
    from paper_2204_01722_amd.binding import PMG
    print_case("vcycle_kept_state", n=n)
    m, H = _hierarchy((n, n, n), (4, 2, 1))
    H.fine.residual(torch.from_numpy(inputs.config1_u(m, amplitude=0.05)).cuda(), store_state=True)
    free = 1.0 - H.masks[0].reshape(-1)
    r = torch.from_numpy((inputs.random_vector(m.n_nodes, 23).reshape(-1) * free).reshape(-1, 3)).cuda()
    out = {}
    for prec in ("f64", "f32"):
        pmg = PMG(H.ops, precision=prec, coarse_fixed_its=8)
        pmg.setup(H.seeds(7))
        out[prec] = t2n(pmg.vcycle(r))
    assert rel(out["f32"], out["f64"]) < 1e-4  # the solver tests' bound for FP32 V-cycles
