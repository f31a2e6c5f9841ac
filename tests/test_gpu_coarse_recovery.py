"""What the one-launch coarse PCG does when a solve does not end in the ordinary way."""
import pytest

from _support import ensure_built, gpu_available, inputs, print_case

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

FACES = {"x0": (1, 1, 1), "x1": (1, 1, 1)}


def _problem(n):
    import torch
    from paper_2204_01722_amd.problem import Hierarchy
    ensure_built()
    m = inputs.box_mesh(n, 2, jitter=0.05, seed=2204)
    H = Hierarchy(m, [2, 1], faces=FACES)
    H.fine.residual(torch.from_numpy(inputs.stretch_field(m, 1.1)).cuda(), store_state=True)
    r = torch.from_numpy(inputs.random_vector(m.n_nodes, 5) * (1.0 - H.masks[0])).cuda()
    return m, H, r


def _pmg(H, **kw):
    from paper_2204_01722_amd.binding import PMG
    pmg = PMG(H.ops, **kw)
    pmg.setup(H.seeds(7))
    return pmg


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_breakdown_on_a_value_that_is_not_finite(precision, value):
    """A right-hand side with one entry that is not finite, near one end of a long bar: the
    coarse solve breaks down at once, and every entry of z that the launch-per-iteration form
    leaves finite or not is so, with the same bits where finite."""
    import numpy as np
    import torch
    print_case("coarse_breakdown", precision=precision, value=value)
    m, H, r = _problem((24, 3, 3))
    r[int(np.argmin(np.abs(m.coords - np.array([0.1, 0.05, 0.05])).sum(axis=1))), 0] = value
    z = _pmg(H, precision=precision, coarse_rtol=1e-3).vcycle(r)
    ref = _pmg(H, precision=precision, coarse_fixed_its=1).vcycle(r)
    assert 0 < int(ref.isfinite().sum()) < ref.numel()
    print(f"  finite entries {int(z.isfinite().sum())}, reference {int(ref.isfinite().sum())} of {ref.numel()}",
          flush=True)
    assert torch.equal(z.isfinite(), ref.isfinite())
    assert torch.equal(z[ref.isfinite()], ref[ref.isfinite()])
