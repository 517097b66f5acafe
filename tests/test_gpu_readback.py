"""Reads of fields and populations to the host: large reads go through shared
pinned slots with helper threads, small ones (and those that find the slots in
use) through plain copies.  Both must give the same bits: a read of one field
of these lattices is small, a read of all of them large."""
import ctypes as C
import threading

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


def _sim(L, lattice, dims, prec, seed=1):
    rng = np.random.default_rng(seed)
    sh = dims[::-1]
    psi = rng.uniform(-0.9, 0.9, sh if lattice == "D3Q19" else (1,) + sh)
    rR, rB = W.colour_densities(psi)
    d = dims if lattice == "D3Q19" else dims[:2] + (1,)
    w = W.Workload("rb", lattice, d, rR, rB, rng.uniform(-0.02, 0.02, (3,) + psi.shape), 1.2, 0.7, 0.01, 0.7)
    s = L.Sim.from_workload(w, precision=prec)
    s.step(3)
    return s


def _read(L, s, wanted):
    """lbcg_fields with only the wanted outputs."""
    n = int(np.prod(s.shape))
    out = {k: np.full((3 if k == "u" else 1) * n, np.nan) for k in wanted}
    p = [out[k].ctypes.data_as(C.POINTER(C.c_double)) if k in out else None for k in ("rhoR", "rhoB", "u", "psi")]
    assert L.load_library().lbcg_fields(s._handle(), *p) == 0
    return out


# node counts around the slot's chunk (8 MiB / 6 rows = 174762 nodes) and not
# multiples of the helpers' shares
@pytest.mark.parametrize("lattice,dims,prec", [("D3Q19", (61, 47, 43), "f32"), ("D3Q19", (56, 56, 56), "f16"),
                                               ("D3Q19", (83, 81, 79), "f32"), ("D2Q9", (701, 499), "f64")])
def test_large_reads_match_small_ones(L, lattice, dims, prec):
    print(f"readback {lattice} {dims} {prec}", flush=True)
    s = _sim(L, lattice, dims, prec)
    f = s.fields()
    for k in ("rhoR", "rhoB", "psi"):
        assert np.array_equal(_read(L, s, [k])[k], f[k].ravel()), k
    some = _read(L, s, ["rhoB", "u"])  # rows in two runs, the others skipped
    assert np.array_equal(some["rhoB"], f["rhoB"].ravel())
    assert np.array_equal(some["u"], f["u"].ravel())
    p = s.populations()
    n = int(np.prod(s.shape))
    nodes = np.unique(np.concatenate([[0, n - 1], np.random.default_rng(2).integers(0, n, 500)]))
    flat = p.reshape(2, p.shape[1], n)
    assert np.array_equal(s.populations_at(nodes), flat[:, :, nodes].transpose(2, 0, 1))
    assert np.allclose(p[0].sum(axis=0), f["rhoR"], rtol=0, atol=1e-5)


def test_reads_on_several_threads(L):
    sims = [_sim(L, "D3Q19", (64, 60, 52), "f32", seed=k) for k in range(4)]
    ref = [s.fields() for s in sims]
    got = [[] for _ in sims]

    def work(j):
        for _ in range(4):
            got[j].append(sims[j].fields())
    th = [threading.Thread(target=work, args=(j,)) for j in range(4)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for j in range(4):
        assert len(got[j]) == 4
        for f in got[j]:
            for k in f:
                assert np.array_equal(f[k], ref[j][k])
    for s in sims:  # the last handle frees the slots; a later one gets new ones
        s.close()
    s = _sim(L, "D3Q19", (64, 60, 52), "f32", seed=0)
    assert np.array_equal(s.fields()["psi"], ref[0]["psi"])
