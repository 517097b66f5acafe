"""The split steps at sizes near their limits: byte offsets just below 2^32, the
largest cubes that the fused kernel takes (304^3 FP32, 383^3 FP16), with the form
chosen by hand and asserted, one step at sampled nodes against the oracle."""
import pytest

from paper_1711_02003_amd import workloads as W
from tests.test_gpu_split import L  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("edge,prec,kernel", [(304, "f32", "FUSED"), (304, "f32", "COMPACT"), (383, "f16", "FUSED"),
                                              (383, "f16", "COMPACT")])
def test_split_largest_lattice_sampled(L, orc, edge, prec, kernel):  # noqa: F811
    from tests.test_gpu_parity import _sampled_one_step
    w = W.droplets_27(L=edge, seed=2)
    s = L.Sim.from_workload(w, precision=prec, kernel=getattr(L, "KERNEL_" + kernel)).set_step_form(L.FORM_SPLIT)
    assert s.step_form() == L.FORM_SPLIT
    s.step(3)
    worst = _sampled_one_step(L, orc, w, s, n_samples=32, seed=edge)
    print(f"split {edge}^3 {prec} {kernel}: sampled one-step max rel diff {worst:.2e}", flush=True)
    # FP16: two units of a stored share, as the sweeps' tests of these sizes
    assert worst < (2e-6 if prec == "f32" else 2 * 2.0 ** -9)
    s.close()
