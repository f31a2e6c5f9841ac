"""The one-launch coarse PCG against the launch-per-iteration one (reached with a fixed
iteration count), and handles on several threads."""
import threading

import pytest

from _support import ensure_built, gpu_available, inputs, print_case

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

FACES = {"x0": (1, 1, 1), "x1": (1, 1, 1)}


def _problem(n, orders):
    import torch
    from paper_2204_01722_amd.problem import Hierarchy
    ensure_built()
    m = inputs.box_mesh(n, orders[0], jitter=0.05, seed=2204)
    H = Hierarchy(m, orders, faces=FACES)
    H.fine.residual(torch.from_numpy(inputs.stretch_field(m, 1.1)).cuda(), store_state=True)
    r = torch.from_numpy(inputs.random_vector(m.n_nodes, 5) * (1.0 - H.masks[0])).cuda()
    return H, r


def _vcycle(H, r, **kw):
    from paper_2204_01722_amd.binding import PMG
    pmg = PMG(H.ops, **kw)
    pmg.setup(H.seeds(7))
    z = pmg.vcycle(r)
    return z, pmg.info(0)[1]


# rows of the coarse level: 72 (a part of one block of 256), 375 (two blocks, one
# workgroup), 648 (two workgroups, a node split between them), 1980, 3993, 27,783 (55
# workgroups, their sums read by two waves) and 52,728 (103, by four)
@pytest.mark.parametrize("n", [(1, 2, 3), (4, 4, 4), (5, 5, 5), (9, 10, 5), (10, 10, 10), (20, 20, 20), (25, 25, 25)])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_one_launch_equals_launch_per_iteration(n, precision):
    """Same iterates bit for bit, and a second solve repeats them."""
    import torch
    print_case("one_launch", n=n, precision=precision)
    H, r = _problem(n, [2, 1])
    z, its = _vcycle(H, r, precision=precision, coarse_rtol=1e-3)
    assert torch.equal(z, _vcycle(H, r, precision=precision, coarse_rtol=1e-3)[0])
    if its == 0:  # no free coarse unknown: nothing to iterate on
        assert n == (1, 2, 3)
        return
    ref, _ = _vcycle(H, r, precision=precision, coarse_fixed_its=its)
    assert torch.equal(z, ref)


@pytest.mark.parametrize("n,precision,layout", [((9, 10, 5), "f64", "nodes"), ((9, 10, 5), "f32", "nodes"),
                                                ((36, 36, 36), "f32", "rows"), ((36, 36, 36), "f32", "nodes"),
                                                ((36, 36, 36), "f64", "rows")])
def test_other_layouts_and_two_rows_a_thread(n, precision, layout):
    """Where the two forms group a sum differently (node-major blocks, and more than 131,072
    rows, which in FP32 take two rows a thread and in FP64 stay launch by launch), a few
    iterations agree to the rounding of the vectors' precision."""
    print_case("one_launch_other", n=n, precision=precision, layout=layout)
    H, r = _problem(n, [2, 1])
    z, its = _vcycle(H, r, precision=precision, coarse_rtol=0.3, coarse_block_layout=layout)
    ref, _ = _vcycle(H, r, precision=precision, coarse_fixed_its=its, coarse_block_layout=layout)
    d = float((z - ref).norm() / ref.norm())
    print(f"  {its} iterations, rel diff {d:.2e}", flush=True)
    assert its > 0 and d <= (1e-12 if precision == "f64" else 1e-5)


def test_iteration_limit():
    """Stops after coarse_maxit iterations with that count."""
    import torch
    H, r = _problem((6, 6, 6), [2, 1])
    z, its = _vcycle(H, r, coarse_rtol=1e-12, coarse_maxit=7)
    assert its == 7 and torch.equal(z, _vcycle(H, r, coarse_fixed_its=7)[0])


def test_handles_on_threads_and_streams():
    """Solves of three handles on three threads and streams, whose launches together exceed
    the device's compute units, give the sequential results."""
    import torch
    from paper_2204_01722_amd.binding import PMG
    cases = []
    for k in range(3):
        H, r = _problem((24, 24, 24), [2, 1])
        pmg = PMG(H.ops, precision="f64")
        pmg.setup(H.seeds(7))
        r = r * (1.0 + k)
        cases.append((H, pmg, r, pmg.vcycle(r)))
    torch.cuda.synchronize()
    bad = []

    def work(k):
        _, pmg, r, ref = cases[k]
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(5):
                if not torch.equal(pmg.vcycle(r), ref):
                    bad.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
