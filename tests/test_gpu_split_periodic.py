"""The split step of periodic D3Q19 lattices (two kernels, one thread per
node), which the automatic launch shape takes on lattices too small to fill
the device with the column sweep.

Every value is formed by the sweep's expressions in the sweep's order, so a
handle on the automatic shape must hold bitwise the state of one whose launch
shape is given (the sweep), on the pair and on the compact state, and on the
pair state the generic kernel's: sizes below and above a block of threads,
planes of exactly one block, widths of one node and of a power of two, and
extents of one, two and three, where a node is its own neighbour."""
import numpy as np
import pytest

from paper_1711_02003_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_02003_amd import lbcg
    lbcg.load_library()
    return lbcg


def _fields(dims, seed):
    nx, ny, nz = dims
    rng = np.random.default_rng(seed)
    psi = np.tanh(np.sin(np.arange(nx)[None, None, :] / 3.0) * 3 + rng.normal(0, 0.3, (nz, ny, nx)))
    rR, rB = W.colour_densities(psi)
    return rR, rB, rng.uniform(-0.02, 0.02, (3, nz, ny, nx))


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("dims", [(5, 7, 6), (1, 9, 20), (16, 16, 2), (64, 4, 3), (257, 1, 1), (33, 17, 9), (70, 45, 11)])
def test_split_periodic_matches_sweep_bitwise(L, dims, prec):
    f = _fields(dims, seed=sum(dims))
    print(f"periodic split {dims} {prec}", flush=True)
    for kernel, others in ((L.KERNEL_FUSED, (dict(kernel=L.KERNEL_FUSED, tile=(8, 1, 0)), dict(kernel=L.KERNEL_GENERIC))),
                           (L.KERNEL_COMPACT, (dict(kernel=L.KERNEL_COMPACT, tile=(8, 1, 64)),))):
        sims = [L.Sim("D3Q19", dims, 1.2, 0.7, 0.01, 0.7, prec, **kw)
                for kw in (dict(kernel=kernel),) + others]
        for s in sims:
            s.init_fields(*f)
        # an odd and an even number of steps, single launches and a replayed
        # graph, with reads of the state (a compact state is expanded) between
        for n in (1, 2, 35):
            for s in sims:
                s.step(n)
            p = sims[0].populations()
            assert np.isfinite(p).all()
            for s in sims[1:]:
                assert np.array_equal(p, s.populations()), (dims, prec, kernel, n)
        # a restored state continues alike
        blob = sims[0].get_state()
        for s in sims:
            s.set_state(blob)
            s.step(3)
        for s in sims[1:]:
            assert np.array_equal(sims[0].populations(), s.populations())
            assert s.diagnostics()["step"] == 41
