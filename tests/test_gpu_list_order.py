"""The node list of the split steps with geometry on lattices whose rows start
on 64-node boundaries, where it goes by tiles of 64 x 8 nodes: heights below,
at and past the tile's, one and several tiles wide, partly filled with walls,
inlets and outlets."""
import numpy as np
import pytest

from tests.test_gpu_split import L, _sparse_geometry  # noqa: F401  (L is a fixture)

pytestmark = pytest.mark.gpu

DIMS = [(64, 1, 9), (64, 7, 3), (64, 8, 2), (128, 9, 4), (192, 17, 3), (320, 24, 2)]


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("dims", DIMS)
def test_tiled_list_matches_sweep_bitwise(L, dims, prec):  # noqa: F811
    w = _sparse_geometry(dims, seed=sum(dims), fluid=0.6, io=min(dims) > 2)
    fl = w.mask == 0
    a, b = (L.Sim.from_workload(w, precision=prec, kernel=L.KERNEL_FUSED) for _ in range(2))
    a.set_step_form(L.FORM_SPLIT)
    b.set_step_form(L.FORM_SWEEP)
    for n in (2, 34):
        pa, pb = (s.step(n).populations()[..., fl] for s in (a, b))
        print(f"tiled list {dims} {prec} {fl.mean():.2f} fluid, {n} steps", flush=True)
        assert np.isfinite(pb).all() and np.array_equal(pa, pb)
    # the lists of the compact state: as the pair state up to rounding
    if prec == "f32":
        c = L.Sim.from_workload(w, precision=prec, kernel=L.KERNEL_COMPACT).step(36)
        pc = c.populations()[..., fl]
        assert np.abs(pc - pb).max() / np.abs(pb).max() < 36 * 4 * 2.0 ** -24
        assert c.diagnostics()["step"] == a.diagnostics()["step"] == 36
