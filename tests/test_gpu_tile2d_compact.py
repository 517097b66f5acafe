"""The D2Q9 compact step against independent paths, in both of its tile shapes
and on ragged lattices: the first step, which reads pairs and stores the compact
state, against the two-pass kernel; the steps after it against the FP64 two-pass
kernel."""
import numpy as np
import pytest

from tests.test_gpu_split import L  # noqa: F401  (a fixture)
from tests.test_gpu_tile2d import _droplets, _random

pytestmark = pytest.mark.gpu

# one tile and less, ragged in both directions, the large tiles (from 800 000 nodes on)
DIMS = [(5, 4), (32, 8), (33, 9), (95, 41), (501, 407), (1003, 811)]


@pytest.mark.parametrize("dims", DIMS)
def test_compact2d_first_steps_match_two_passes(L, dims):  # noqa: F811
    # Step 1 runs the two passes, step 2 reads pairs and stores the compact
    # state: total deviations of step 2 are formed by the same expressions, and
    # the shares differ by the rounding of the receiver's split.
    w = _random(dims, seed=sum(dims))
    a = L.Sim.from_workload(w, precision="f32", kernel=L.KERNEL_COMPACT).step(2)
    g = L.Sim.from_workload(w, precision="f32", kernel=L.KERNEL_GENERIC).step(2)
    assert a.step_form() == L.FORM_TILE and g.step_form() == L.FORM_TWO_PASS
    pa, pg = a.populations(), g.populations()
    d = float(np.abs(pa - pg).max() / np.abs(pg).max())
    t = float(np.abs(pa.sum(0) - pg.sum(0)).max() / np.abs(pg).max())
    print(f"compact2d {dims}: colours {d:.2e}, totals {t:.2e} after 2 steps", flush=True)
    # totals: the export rounds each colour to FP32 of a share once (2^-24 of a
    # population twice); colours: the share's own rounding, at most four units
    assert t < 2 * 2.0 ** -24
    assert d < 4 * 2.0 ** -23


@pytest.mark.parametrize("dims", DIMS)
def test_compact2d_matches_f64_two_passes(L, dims):  # noqa: F811
    w = _droplets(dims, seed=sum(dims))
    a = L.Sim.from_workload(w, precision="f32", kernel=L.KERNEL_COMPACT).step(40)
    g = L.Sim.from_workload(w, precision="f64", kernel=L.KERNEL_GENERIC).step(40)
    pa, pg = a.populations(), g.populations()
    d = float(np.abs(pa - pg).max() / np.abs(pg).max())
    print(f"compact2d {dims} x40 against FP64: {d:.2e}", flush=True)
    assert d < 40 * 4 * 2.0 ** -23
