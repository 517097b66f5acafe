"""Batched split D3Q19 steps: one launch of each kernel over many lattices.

Lattices narrower than a sweep tile, where the batched launches take the split
step: their node counts leave a last block partly filled (and one lattice of
fewer nodes than a block, one with no fluid at all), and they stop at different
steps, so the block map shrinks.  Each lattice must come out bitwise as stepped
alone, which other tests hold against the generic kernel and the oracle.
"""
import numpy as np
import pytest

from paper_1711_02003_amd import workloads as W
from tests.test_gpu_split import L, _sparse_geometry  # noqa: F401  (L is a fixture)

pytestmark = pytest.mark.gpu


def _box(dims, seed):
    rng = np.random.default_rng(seed)
    sh = dims[::-1]
    psi = np.tanh(np.sin(np.arange(dims[0])[None, None, :] / 3.0) * 3 + rng.normal(0, 0.3, sh))
    rR, rB = W.colour_densities(psi)
    return W.Workload(f"box{dims}", "D3Q19", dims, rR, rB, rng.uniform(-0.02, 0.02, (3,) + sh), 1.2, 0.7, 0.01, 0.7)


def _walls(dims):
    sh = dims[::-1]
    return W.Workload("walls", "D3Q19", dims, np.full(sh, 0.6), np.full(sh, 0.4), None, 1.0, 0.8, 0.01, 0.7,
                      mask=np.ones(sh, np.uint8))


@pytest.mark.parametrize("prec", ["f32", "f16"])
@pytest.mark.parametrize("state", ["pairs", "compact"])
def test_batched_split_matches_alone_bitwise(L, prec, state):  # noqa: F811
    import torch
    ws = [_box((20, 17, 13), 1), _box((5, 4, 3), 2), _box((16, 16, 16), 3)]
    if state == "pairs":  # the batched compact state is periodic only
        ws += [_sparse_geometry((24, 13, 9), 4), _sparse_geometry((6, 5, 7), 5), _walls((8, 4, 3))]
    kern = L.KERNEL_FUSED if state == "pairs" else L.KERNEL_COMPACT
    stream = torch.cuda.Stream()
    sims = [L.Sim.from_workload(w, precision=prec, kernel=kern, stream=stream.cuda_stream) for w in ws]
    steps = [41, 3, 36, 41, 2, 37][: len(ws)]
    for s in sims:  # compact lattices start from pairs: the first step alone
        s.step(1)
    b = L.Batch(sims)
    b.step(steps)  # replays a graph of 32 levels
    b.close()
    L.batch_step_noalloc(sims, [4, 0, 1, 5, 2, 3][: len(ws)], (8, 8))
    for w, s, n, m in zip(ws, sims, steps, [4, 0, 1, 5, 2, 3]):
        print(f"batched split {state} {prec} {w.dims}", flush=True)
        ref = L.Sim.from_workload(w, precision=prec, kernel=kern)
        ref.step(1 + n + m)
        fl = slice(None) if w.mask is None else w.mask == 0
        assert np.array_equal(s.populations()[..., fl], ref.populations()[..., fl])
        assert s.diagnostics()["step"] == 1 + n + m
        ref.close()
    for s in sims:
        s.close()
