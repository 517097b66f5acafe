"""The D2Q9 tile step at the sizes where it can go wrong: both of its tile
shapes on ragged lattices (the large tiles serve lattices of about a million
nodes on, with geometry of four million), in every storage and collision form
it takes, bitwise the two-pass generic kernel; FP64, which the generic kernel
no longer steps, against the oracle; the compact state on the large tiles
against the small ones."""
import numpy as np
import pytest

from paper_1711_02003_amd import workloads as W
from tests.helpers import oracle_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_02003_amd import lbcg
    lbcg.load_library()
    return lbcg


def _random(dims, seed, masked=False):
    rng = np.random.default_rng(seed)
    nx, ny = dims
    sh = (1, ny, nx)
    u = np.zeros((3,) + sh)
    u[:2] = rng.uniform(-0.04, 0.04, (2,) + sh)
    w = W.Workload("random2d", "D2Q9", (nx, ny, 1), rng.uniform(0.05, 1, sh), rng.uniform(0.05, 1, sh), u, 1.3, 0.7,
                   0.01, 0.7)
    if masked:
        m = np.zeros(sh, np.uint8)
        m[:, 0], m[:, -1] = 1, 64  # a neutral and a wetting wall
        m[:, 1:-1, 0], m[:, 1:-1, -1] = 2, 128
        m[0, ny // 2, nx // 2] = 1
        w.mask = m
        w.inlets = [{"u": (0.01, 0.002, 0.0), "rho_R": 0.8, "rho_B": 0.2}]
        w.outlets = [{"rho": 1.02}]
        w.walls = [{"psi": 0.4}]
    return w


def _droplets(dims, seed):
    # FP16 storage with plain BGK needs the shares of a smooth field
    w = _random(dims, seed)
    nx, ny = dims
    x, y = np.arange(nx)[None, None, :], np.arange(ny)[None, :, None]
    w.rhoR, w.rhoB = W.colour_densities(np.tanh(3 * np.sin(x / 9.0) * np.cos(y / 7.0)))
    w.u = w.u * 0.05
    return w


@pytest.mark.parametrize("prec,coll", [("f32", "REGULARIZED"), ("f16", "REGULARIZED"), ("f32", "BGK"),
                                       ("f32", "BGK_COLOUR"), ("f16", "BGK")])
def test_large_tiles_match_generic_bitwise(L, prec, coll):
    w = _droplets((1003, 811), seed=5)
    sims = [L.Sim.from_workload(w, precision=prec, kernel=k, collision=getattr(L, coll))
            for k in (L.KERNEL_FUSED, L.KERNEL_GENERIC)]
    fields = []
    for s in sims:
        s.step(7)
        fields.append(s.populations())
        s.close()
    print(f"large tiles {prec} {coll}", flush=True)
    assert np.isfinite(fields[0]).all()
    assert np.array_equal(*fields)


@pytest.mark.parametrize("prec", ["f32", "f16"])
def test_large_tiles_with_geometry_match_generic_bitwise(L, prec):
    w = W.flow_focusing_2d(4100, 1000, u_disp=0.02, u_side=0.03)
    fl = w.mask == 0
    fields = []
    for k in (L.KERNEL_FUSED, L.KERNEL_GENERIC):
        s = L.Sim.from_workload(w, precision=prec, kernel=k)
        s.step(9)
        fields.append({n: v[..., fl] for n, v in s.fields().items()})
        s.close()
    for n in fields[0]:
        assert np.array_equal(fields[0][n], fields[1][n]), n


@pytest.mark.parametrize("kernel", ["KERNEL_COMPACT", "KERNEL_FUSED"])
def test_large_tiles_match_small_tiles_bitwise(L, kernel):
    # 2 x 2 copies of a periodic field step like the field itself; the copies
    # are large enough for the large tiles, the field for the small ones
    w = _random((501, 407), seed=6)
    s = L.Sim.from_workload(w, precision="f32", kernel=getattr(L, kernel)).step(12)
    one = s.populations()
    w4 = W.Workload("copies", "D2Q9", (1002, 814, 1), np.tile(w.rhoR, (1, 2, 2)), np.tile(w.rhoB, (1, 2, 2)),
                    np.tile(w.u, (1, 1, 2, 2)), w.tau_R, w.tau_B, w.A, w.beta)
    t = L.Sim.from_workload(w4, precision="f32", kernel=getattr(L, kernel)).step(12)
    assert np.array_equal(t.populations(), np.tile(one, (1, 1, 1, 2, 2)))


@pytest.mark.parametrize("dims", [(5, 4), (1, 40), (40, 1), (33, 9), (64, 8), (65, 17)])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("coll", ["REGULARIZED", "BGK"])
def test_f64_tiles_match_oracle(L, orc, dims, masked, coll):
    if masked and min(dims) < 4:
        pytest.skip("the walls would leave no fluid node")
    w = _random(dims, seed=sum(dims), masked=masked)
    s = L.Sim.from_workload(w, precision="f64", collision=getattr(L, coll)).step(60)
    o = orc.Oracle(oracle_params(orc, w, collision=getattr(orc, coll))).init(w.rhoR, w.rhoB, w.u).step(60)
    fl = np.ones(w.shape, bool) if w.mask is None else w.mask == 0
    a, b = s.populations()[..., fl], o.populations()[..., fl]
    d = float(np.abs(a - b).max() / np.abs(b).max())
    print(f"f64 tiles {dims} masked={masked} {coll}: {d:.2e}", flush=True)
    assert d < 1e-12
