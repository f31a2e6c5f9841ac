"""The adjoint with more quadrature points than nodes in a direction, and adjoint and diagonal
where the elements fill the workgroups' tiles exactly or fall one short."""
import numpy as np
import pytest

from _support import ensure_built, gpu_available, inputs, print_case, rel, t2n

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

TOL = {"f64": 1e-12, "f32": 1e-5}  # those of the operator tests


def _check(p, q, n, mode):
    import torch
    from oracle import fem
    from paper_2204_01722_amd.problem import Hierarchy
    ensure_built()
    print_case("adjoint_forms", p=p, q=q, n=n, mode=mode)
    mu_e, lam_e = inputs.loguniform_materials(int(np.prod(n)), seed=4)
    m = inputs.box_mesh(n, p, jitter=0.05, seed=2204)
    H = Hierarchy(m, [p], faces={"x0": (1, 0, 1)}, mu_e=mu_e, lam_e=lam_e, q=q)
    op, mask = H.fine, H.masks[0]
    u, w = inputs.config1_u(m, amplitude=0.05), inputs.random_vector(m.n_nodes, 5)
    ut, wt = torch.from_numpy(u).cuda(), torch.from_numpy(w).cuda()
    op.residual(ut, store_state=True)
    op.state_cast_f32()
    d = fem.make_disc(m.coords, m.elem_nodes, p + 1, q)
    ref = fem.residual_vjp(d, u, w, mu_e, lam_e, mask)
    diag = fem.diagonal(d, u, mu_e, lam_e, mask)
    for prec in ("f64", "f32"):
        ww = wt if prec == "f64" else wt.float()
        for got, r in zip(op.residual_vjp(ut, ww, mode=mode, precision=prec), ref):
            assert rel(t2n(got), r) < TOL[prec]
        alone = op.residual_vjp(ut, ww, mode=mode, precision=prec, want_params=False)[0]
        assert rel(t2n(alone), ref[0]) < TOL[prec]
        assert rel(t2n(op.diagonal(prec)), diag) < TOL[prec]


# every instantiated pair of more points than nodes; tiles of 9, 1, 2 and 1 elements
@pytest.mark.parametrize("p, q", [(1, 3), (1, 4), (1, 5), (2, 4), (2, 5), (3, 5), (4, 6)])
@pytest.mark.parametrize("mode", ["stored", "recompute"])
def test_more_points_than_nodes(p, q, mode):
    for n in [(1, 1, 1), (3, 1, 1), (8, 1, 1), (3, 3, 1), (5, 2, 1)]:
        _check(p, q, n, mode)


# two points: tiles of 32 elements; three points: tiles of 9
@pytest.mark.parametrize("p, n", [(1, (31, 1, 1)), (1, (8, 2, 2)), (1, (3, 11, 1)), (1, (4, 4, 4)), (2, (8, 1, 1)),
                                  (2, (3, 3, 1)), (2, (6, 3, 1))])
@pytest.mark.parametrize("mode", ["stored", "recompute"])
def test_full_tiles(p, n, mode):
    _check(p, p + 1, n, mode)
