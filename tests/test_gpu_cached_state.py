"""Inside a V-cycle a linearisation that fits the last-level cache is loaded with plain loads,
by any other action with nontemporal ones: the same bits either way."""
import pytest

from _support import ensure_built, gpu_available, inputs, print_case

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# states of 77 MiB (FP64, 17^3) and 122 MiB (FP32, 25^3) take the plain loads, the last tile
# ragged; those of 8^3 elements (8 and 4 MiB) take the nontemporal ones on both sides
@pytest.mark.parametrize("n, precision", [(17, "f64"), (25, "f32"), (8, "f64"), (8, "f32")])
def test_smoothing_equals_single_actions(n, precision):
    """With every coarse component constrained the correction is zero, and with one step a
    sweep z = x + D^-1 (r - A x) / theta, x = D^-1 r / theta, each operation rounded once."""
    import numpy as np
    import torch
    from paper_2204_01722_amd.binding import PMG, Operator
    from paper_2204_01722_amd.problem import Hierarchy
    ensure_built()
    print_case("cached_state", n=n, precision=precision)
    m = inputs.box_mesh(n, 4, jitter=0.05, seed=2204)
    H = Hierarchy(m, [4], faces={"x0": (1, 1, 1)})
    op = H.fine
    nc = (2 * n + 1) ** 3
    topo = torch.from_numpy(np.ascontiguousarray(inputs.box_topology(m.n, 2), np.int32)).cuda()
    coarse = Operator(3, 5, topo, nc, torch.ones(nc, 3, dtype=torch.uint8, device="cuda"), fine=op)
    op.residual(torch.from_numpy(inputs.config1_u(m, amplitude=0.05)).cuda(), store_state=True)
    pmg = PMG([op, coarse], precision=precision, cheb_degree=1)
    pmg.setup([torch.from_numpy(inputs.rough_seed(m.n_nodes, H.masks[0], 7)).cuda()])
    dt = torch.float64 if precision == "f64" else torch.float32
    r = torch.from_numpy(inputs.random_vector(m.n_nodes, 23) * (1.0 - H.masks[0])).cuda()
    z = pmg.vcycle(r)
    lam = pmg.info(0)[0]
    c = 1.0 / (0.5 * (pmg.params.cheb_hi * lam + pmg.params.cheb_lo * lam))
    b, dinv = r.to(dt), 1.0 / op.diagonal(precision)
    x = dinv * b * c
    x = x + dinv * (b - op.jacobian(x, precision)) * c
    assert torch.equal(z, x.double())
