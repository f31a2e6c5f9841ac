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


# 27,783 rows in 55 workgroups, 375 in one (which waits for nobody), 151,959 in FP32 (149
# workgroups of two rows a thread) and in FP64, where they do not fit
@pytest.mark.parametrize("n, precision, one_launch", [(20, "f64", 1), (20, "f32", 1), (4, "f64", 1), (36, "f32", 1),
                                                      (36, "f64", 0)])
def test_which_form_made_the_solve(n, precision, one_launch):
    print_case("coarse_form", n=n, precision=precision)
    _, H, r = _problem((n, n, n))
    pmg = _pmg(H, precision=precision, coarse_rtol=0.1)
    pmg.vcycle(r)
    assert pmg.coarse_stats() == {"one_launch": one_launch, "launches": 1 - one_launch, "given_up": 0}


@pytest.mark.parametrize("n, precision", [(20, "f64"), (20, "f32"), (36, "f32")])
def test_a_solve_given_up_is_made_again(n, precision):
    """With no patience at all the workgroups give up at their first look; the solve that
    launches make instead starts from the same right-hand side.  After 32 more of those one
    launch is tried again, and after a second loss in a row 64."""
    import torch
    from paper_2204_01722_amd.binding import HpmgError
    print_case("coarse_given_up", n=n, precision=precision)
    _, H, r = _problem((n, n, n))
    kw = dict(precision=precision, coarse_rtol=0.1 if n == 36 else 1e-3)
    pmg = _pmg(H, **kw)
    ref = pmg.vcycle(r)
    its = pmg.info(0)[1]

    def same(z):
        if n == 36:  # two rows a thread group the sums otherwise than the launches do
            return float((z - ref).norm() / ref.norm()) <= 1e-5
        return torch.equal(z, ref)

    pmg.set_coarse_wait(0.0)
    assert same(pmg.vcycle(r)) and pmg.info(0)[1] == its
    assert pmg.coarse_stats() == {"one_launch": 1, "launches": 1, "given_up": 1}
    for k in range(32):
        assert same(pmg.vcycle(r))
    assert pmg.coarse_stats() == {"one_launch": 1, "launches": 33, "given_up": 1}
    assert same(pmg.vcycle(r))
    assert pmg.coarse_stats() == {"one_launch": 1, "launches": 34, "given_up": 2}
    pmg.set_coarse_wait(0.1)
    for k in range(64):
        pmg.vcycle(r)
    assert pmg.coarse_stats()["launches"] == 98
    assert torch.equal(pmg.vcycle(r), ref)
    assert pmg.coarse_stats() == {"one_launch": 2, "launches": 98, "given_up": 2}
    for bad in (-1.0, 11.0, float("nan")):
        with pytest.raises(HpmgError):
            pmg.set_coarse_wait(bad)


def test_solves_of_several_threads_all_end():
    """Three handles on three threads and streams, whose launches together exceed the device's
    compute units: every solve ends without an error, with the sequential result, and is made
    in one launch or, where it was not let in or gave up, by launches."""
    from concurrent.futures import ThreadPoolExecutor
    import torch
    cases = []
    for k in range(3):
        _, H, r = _problem((24, 24, 24))
        pmg = _pmg(H, precision="f64")
        r = r * (1.0 + k)
        cases.append((pmg, r, pmg.vcycle(r), H))
    torch.cuda.synchronize()

    def work(k):
        pmg, r, ref, _ = cases[k]
        with torch.cuda.stream(torch.cuda.Stream()):
            return sum(torch.equal(pmg.vcycle(r), ref) for _ in range(5))

    with ThreadPoolExecutor(3) as pool:
        jobs = [pool.submit(work, k) for k in range(3)]
        assert [j.result(timeout=60) for j in jobs] == [5, 5, 5]
    for pmg, *_ in cases:
        st = pmg.coarse_stats()
        assert st["one_launch"] + st["launches"] == 6 and st["one_launch"] > 0
