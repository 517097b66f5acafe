"""The forms of the batched steps: sweep and split step for the periodic and for
the geometry lattices, each chosen by hand and asserted, in lbcg_batch_step
(single levels and replayed graphs) and in lbcg_batch_step_noalloc.  Each lattice
must come out bitwise as stepped alone."""
import numpy as np
import pytest

from tests.test_gpu_split import L, _sparse_geometry  # noqa: F401  (L is a fixture)
from tests.test_gpu_split_batch import _box

pytestmark = pytest.mark.gpu

FORMS = [("SWEEP", "SWEEP"), ("SPLIT", "SPLIT"), ("SWEEP", "SPLIT"), ("SPLIT", "SWEEP")]


def _workloads(state):
    # wider than a tile, ragged, and smaller than a block of threads
    ws = [_box((70, 17, 13), 1), _box((5, 4, 3), 2), _box((16, 16, 16), 3)]
    if state == "pairs":
        ws += [_sparse_geometry((67, 13, 9), 4, io=False), _sparse_geometry((24, 9, 7), 5)]
    return ws


def _sims(L, ws, prec, state):  # noqa: F811
    import torch
    stream = torch.cuda.Stream()
    kern = L.KERNEL_FUSED if state == "pairs" else L.KERNEL_COMPACT
    sims = [L.Sim.from_workload(w, precision=prec, kernel=kern, stream=stream.cuda_stream) for w in ws]
    for s in sims:
        s._torch_stream = stream
    return sims


def _check(L, ws, sims, steps, prec, state, what):  # noqa: F811
    kern = L.KERNEL_FUSED if state == "pairs" else L.KERNEL_COMPACT
    for w, s, n in zip(ws, sims, steps):
        ref = L.Sim.from_workload(w, precision=prec, kernel=kern)
        ref.step(n)
        fl = slice(None) if w.mask is None else w.mask == 0
        a, b = s.populations()[..., fl], ref.populations()[..., fl]
        assert np.isfinite(b).all()
        assert np.array_equal(a, b), (what, prec, state, w.dims)
        assert s.diagnostics()["step"] == n
        ref.close()


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("state,forms", [("pairs", f) for f in FORMS] + [("compact", f) for f in FORMS[:2]])
def test_batch_in_chosen_forms_matches_alone_bitwise(L, prec, state, forms):  # noqa: F811
    ws = _workloads(state)
    sims = _sims(L, ws, prec, state)
    p, g = (getattr(L, "FORM_" + f) for f in forms)
    want = (p, g if state == "pairs" else L.FORM_AUTO)
    b = L.Batch(sims, tile=(8, 4))
    assert b.step_form() == (L.FORM_SWEEP, L.FORM_SWEEP if state == "pairs" else L.FORM_AUTO)  # a given tile
    n1 = [36, 3, 35, 36, 34][: len(ws)]
    b.set_step_form(p, g)
    assert b.step_form() == want == b.launch_info()["forms"]
    b.step(n1)  # replays a graph of 32 levels
    # the other forms, then these again (graphs made anew), other counts
    q, h = (L.FORM_SPLIT + L.FORM_SWEEP - f for f in (p, g))
    b.set_step_form(q, h).step([2, 1, 33, 0, 5][: len(ws)])
    assert b.set_step_form().step_form()[0] == L.FORM_SWEEP  # the batch's own choice
    b.set_step_form(p, g).step([1, 2, 3, 4, 0][: len(ws)])
    total = [x + y + z for x, y, z in zip(n1, [2, 1, 33, 0, 5], [1, 2, 3, 4, 0])]
    b.close()
    print(f"batch forms {forms} {prec} {state}", flush=True)
    _check(L, ws, sims, total, prec, state, forms)


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("tile", [(8, 4), (4, 5)])
@pytest.mark.parametrize("state,forms", [("pairs", f) for f in FORMS] + [("compact", f) for f in FORMS[:2]])
def test_noalloc_in_chosen_forms_matches_alone_bitwise(L, prec, state, forms, tile):  # noqa: F811
    if state == "compact":
        tile = (8, tile[1])
    ws = _workloads(state)
    sims = _sims(L, ws, prec, state)
    p, g = (getattr(L, "FORM_" + f) for f in forms)
    for w, s in zip(ws, sims):
        s.set_step_form(p if w.mask is None else g)
    assert L.batch_noalloc_form(sims, tile) == (p, g if state == "pairs" else L.FORM_AUTO)
    n = [7, 3, 5, 6, 4][: len(ws)]
    L.batch_step_noalloc(sims, n, tile)
    m = [0, 4, 2, 5, 1][: len(ws)]
    L.batch_step_noalloc(sims, m, tile)  # lattices drop out, other counts
    print(f"noalloc forms {forms} {tile} {prec} {state}", flush=True)
    _check(L, ws, sims, [a + b for a, b in zip(n, m)], prec, state, forms)
    # one handle set to the sweep decides for its group
    sims[0].set_step_form(L.FORM_SWEEP)
    assert L.batch_noalloc_form(sims, tile)[0] == L.FORM_SWEEP


def test_timed_choice_is_carried_over(L):  # noqa: F811
    ws = _workloads("pairs")
    sims = _sims(L, ws, "f32", "pairs")
    b = L.Batch(sims)
    i = b.launch_info()
    c = L.Batch(sims, tile=(i["rows"], i["zplanes"])).set_step_form(*i["forms"])
    assert c.launch_info() == i
    # and chosen by hand on a timed batch, and back
    for f in (L.FORM_SWEEP, L.FORM_SPLIT):
        assert b.set_step_form(f, f).step_form() == (f, f)
    assert b.set_step_form().launch_info() == i
    b.close()
    c.close()


def test_refused_forms(L):  # noqa: F811
    w = _box((5, 4, 3), 2)
    sims = _sims(L, [w] * 257, "f32", "pairs")
    b = L.Batch(sims, tile=(8, 4))
    for bad in ((L.FORM_SPLIT, 0), (L.FORM_TILE, 0), (0, -1)):
        with pytest.raises(L.LbcgError) as e:
            b.set_step_form(*bad)
        assert e.value.status == L.E_INVAL
    assert b.step_form() == (L.FORM_SWEEP, L.FORM_AUTO)
    b.close()
    with pytest.raises(L.LbcgError):
        L.batch_noalloc_form(sims, (8, 4))
    with pytest.raises(L.LbcgError):
        L.batch_noalloc_form(sims[:2], (6, 4))
    for s in sims:
        s.close()


def test_noalloc_weighs_the_given_shape(L):  # noqa: F811
    # Groups where the faster form is several times faster or depends on the
    # given launch shape: 128^3 lattices sweep well in chunks of 16 planes (112
    # us against 151) and badly in chunks of 64 (320 against 151), junctions on
    # sweeps take 94 to 381 us against 28.
    from paper_1711_02003_amd import workloads as W
    for kern, w, tile, form in [("COMPACT", W.static_droplet_3d(n=128, R=20.0), (8, 16), "SWEEP"),
                                ("COMPACT", W.static_droplet_3d(n=128, R=20.0), (8, 64), "SPLIT"),
                                ("FUSED", W.static_droplet_3d(n=128, R=20.0), (8, 64), "SPLIT"),
                                ("FUSED", W.flow_focusing(128, 48, 14), (8, 32), "SPLIT"),
                                ("FUSED", _box((20, 17, 13), 1), (4, 4), "SPLIT")]:
        s = L.Sim.from_workload(w, kernel=getattr(L, "KERNEL_" + kern))
        got = L.batch_noalloc_form([s], tile)[0 if w.mask is None else 1]
        print(kern, w.dims, tile, got, flush=True)
        assert got == getattr(L, "FORM_" + form), (kern, w.dims, tile)
        s.close()


def test_timed_compact_batch_keeps_the_faster_form(L):  # noqa: F811
    # one 128^3 lattice, FP16 compact: the sweep takes 93 us a level, the split
    # step 107, and 20 % less than that when a level is timed on a fixed state
    from paper_1711_02003_amd import workloads as W
    s = L.Sim.from_workload(W.static_droplet_3d(n=128, R=20.0), precision="f16", kernel=L.KERNEL_COMPACT).step(2)
    b = L.Batch([s])
    assert b.step_form() == (L.FORM_SWEEP, L.FORM_AUTO)
    b.close()


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("before", [0, 1])
def test_compact_batch_of_fresh_lattices_is_timed_on_their_state(L, prec, before):  # noqa: F811
    # lattices that have not taken their first compact step, in device memory
    # full of NaN: the timing works on compact states made from theirs (here
    # seen in the handle's memory: two pair buffers, then the compact ones),
    # and neither the states nor what follows change
    import torch
    w = _box((20, 17, 13), 1)
    kw = dict(precision=prec, kernel=L.KERNEL_COMPACT)
    n = L.Sim.from_workload(w, **kw).footprint
    mem = torch.full((n + 256,), 255, dtype=torch.uint8, device="cuda")
    ofs = -mem.data_ptr() % 256
    stream = torch.cuda.current_stream().cuda_stream
    s = L.Sim.from_workload(w, dev_buf=(mem.data_ptr() + ofs, n), stream=stream or None, **kw).step(before)
    p = s.populations()
    b = L.Batch([s])
    s.synchronize()
    E, dt = (4, torch.float32) if prec == "f32" else (2, torch.float16)
    pitch = -(-w.nodes // 64) * 64
    at = ofs + 2 * (-(-38 * pitch * E // 256) * 256)
    got = 0
    for k in range(2):
        c = mem[at:at + 19 * pitch * E].view(dt).reshape(19, pitch)[:, :w.nodes]
        got += bool(torch.isfinite(c).all())
        at += -(-(pitch * (19 * E + (20 if E == 4 else 12))) // 256) * 256
    print(f"compact states written by the timing {prec} after {before} steps: {got}", flush=True)
    assert got == 2
    assert np.array_equal(p, s.populations())
    b.step(35)
    b.close()
    ref = L.Sim.from_workload(w, **kw).step(before + 35)
    assert np.array_equal(s.populations(), ref.populations())
    s.close()
