"""Which step a handle runs: its report, its choice, and carrying a tuned choice
over to other handles.  Every form that a handle can take gives bitwise the
same states, also when it changes on the way."""
import numpy as np
import pytest

from paper_1711_02003_amd import workloads as W
from tests.test_gpu_split import L, _sparse_geometry  # noqa: F401  (L is a fixture)
from tests.test_gpu_split_batch import _box

pytestmark = pytest.mark.gpu


def _shape(info):
    return (info["rows"], info["zchunks"], info["tile_width"])


def _full_geometry(dims):
    # a wall on one side only: mostly fluid
    w = _box(dims, 9)
    w.mask = np.zeros(dims[::-1], np.uint8)
    w.mask[:, 0] = 1
    return w


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("state", ["pairs", "compact", "sparse", "full"])
def test_forms_agree_and_can_be_chosen(L, prec, state):  # noqa: F811
    w = {"sparse": _sparse_geometry((24, 13, 9), 4, io=False), "full": _full_geometry((24, 13, 9))}.get(state, _box((24, 13, 9), 3))
    kern = L.KERNEL_COMPACT if state == "compact" else L.KERNEL_FUSED
    fl = slice(None) if w.mask is None else w.mask == 0
    auto = {"full": L.FORM_SWEEP}.get(state, L.FORM_SPLIT)
    sims = [L.Sim.from_workload(w, precision=prec, kernel=kern) for _ in range(3)]
    sims[1].set_step_form(L.FORM_SWEEP)
    sims[2].set_step_form(L.FORM_SPLIT)
    assert [s.launch_info()["form"] for s in sims] == [auto, L.FORM_SWEEP, L.FORM_SPLIT]
    for n in (1, 36, 3):  # single steps and replayed graphs
        for s in sims:
            s.step(n)
    p = sims[0].populations()[..., fl]
    assert np.isfinite(p).all()
    for s in sims[1:]:
        assert np.array_equal(p, s.populations()[..., fl]), (state, prec)
    # the forms change places on the way (the graphs are made again)
    sims[1].set_step_form(L.FORM_SPLIT)
    sims[2].set_step_form(L.FORM_SWEEP)
    for s in sims:
        s.step(35)
    p = sims[0].populations()[..., fl]
    for s in sims[1:]:
        assert np.array_equal(p, s.populations()[..., fl]), (state, prec)
    # tuning keeps to a chosen form; without one it chooses
    assert sims[1].tune()["form"] == L.FORM_SPLIT
    assert sims[2].tune()["form"] == L.FORM_SWEEP
    assert sims[2].set_step_form(L.FORM_AUTO).step_form() == L.FORM_SWEEP  # as tuned
    shape = sims[0].tune()
    assert shape["form"] in (L.FORM_SWEEP, L.FORM_SPLIT)
    # a tuned choice carried over to another handle: the same step in the same shape
    for s in sims:
        info = s.launch_info()
        print(f"step form {state} {prec}: {info}", flush=True)
        t = L.Sim.from_workload(w, precision=prec, kernel=kern, tile=_shape(info)).set_step_form(info["form"])
        assert t.launch_info() == info
        t.step(75)
        assert np.array_equal(p, t.populations()[..., fl]), (state, prec)
        t.close()


def test_given_shape_runs_the_sweep(L):  # noqa: F811
    w = _box((24, 13, 9), 3)
    for kern in (L.KERNEL_FUSED, L.KERNEL_COMPACT):
        s = L.Sim.from_workload(w, kernel=kern, tile=(8, 2, 0))
        assert s.step_form() == L.FORM_SWEEP and _shape(s.launch_info()) == (8, 2, 64)
        assert s.set_step_form(L.FORM_SPLIT).step_form() == L.FORM_SPLIT
        assert s.set_step_form(L.FORM_AUTO).step_form() == L.FORM_SWEEP


def test_forms_that_a_handle_cannot_take_are_refused(L):  # noqa: F811
    w3, g3 = _box((24, 13, 9), 3), _sparse_geometry((24, 13, 9), 4)
    w2 = W.static_droplet_2d(n=32, R=8.0)
    cases = [(L.Sim.from_workload(w3, collision=L.BGK), L.FORM_SWEEP, [L.FORM_SPLIT, L.FORM_TILE]),
             (L.Sim.from_workload(g3, kernel=L.KERNEL_COMPACT), L.FORM_SPLIT, [L.FORM_SWEEP]),
             (L.Sim.from_workload(w3, precision="f64"), L.FORM_TWO_PASS, [L.FORM_SWEEP, L.FORM_SPLIT]),
             (L.Sim.from_workload(w3, kernel=L.KERNEL_GENERIC), L.FORM_TWO_PASS, [L.FORM_SPLIT]),
             (L.Sim.from_workload(w2), L.FORM_TILE, [L.FORM_SWEEP, L.FORM_SPLIT, L.FORM_TWO_PASS]),
             (L.Sim.from_workload(w2, kernel=L.KERNEL_COMPACT), L.FORM_TILE, [L.FORM_SPLIT]),
             (L.Sim.from_workload(w2, precision="f64"), L.FORM_TILE, [L.FORM_TWO_PASS])]
    for s, form, refused in cases:
        assert s.step_form() == form
        for f in refused + [5, -1]:
            with pytest.raises(L.LbcgError) as e:
                s.set_step_form(f)
            assert e.value.status == L.E_INVAL
            assert s.step_form() == form
        assert s.set_step_form(form).step_form() == form


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("coll", ["REGULARIZED", "BGK", "BGK_COLOUR"])
@pytest.mark.parametrize("dims", [(33, 9), (65, 17), (200, 130)])
def test_f64_d2q9_tiles_match_the_two_passes_bitwise(L, dims, coll, masked):  # noqa: F811
    # the automatic choice steps on tiles; a caller that asks for the generic
    # kernel gets the two passes, and both the same bits
    from tests.test_gpu_tile2d import _random
    w = _random(dims, seed=sum(dims), masked=masked)
    fl = slice(None) if w.mask is None else w.mask == 0
    a = L.Sim.from_workload(w, precision="f64", collision=getattr(L, coll))
    g = L.Sim.from_workload(w, precision="f64", collision=getattr(L, coll), kernel=L.KERNEL_GENERIC)
    assert a.launch_info()["kernel"] == g.launch_info()["kernel"] == L.KERNEL_GENERIC
    assert a.step_form() == L.FORM_TILE and g.step_form() == L.FORM_TWO_PASS
    for n in (1, 2, 35):
        p, q = (s.step(n).populations()[..., fl] for s in (a, g))
        assert np.isfinite(p).all() and np.array_equal(p, q), (dims, coll, masked, n)
