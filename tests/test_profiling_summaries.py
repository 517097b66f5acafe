"""The summaries of kernel traces report timed regions only: a kernel that ran
as a tuner's trials and was not picked has no row."""
import csv

import pytest

from paper_1711_02003_amd import profiling

SWEEP = "_ZN4lbcg12_GLOBAL__N_112k_step_fusedIDF16_fLi8ELb0ELb0EEEvNS_9FusedArgsIT_EE"
MOMENTS = "_ZN4lbcg12_GLOBAL__N_115k_split_momentsIDF16_Lb0ELb0EEEvNS_9SplitDescE"
COLLIDE = "_ZN4lbcg12_GLOBAL__N_115k_split_collideIDF16_Lb0EEEvNS_9SplitDescE"
PAIRS = "void lbcg::(anonymous namespace)::k_step_fused<float, float, 8, false, false>(lbcg::FusedArgs<float>)"


def _trace(path, launches):
    """launches: (kernel, grid, duration us), one after another."""
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Kernel_Name", "Start_Timestamp", "End_Timestamp", "Grid_Size_X", "Workgroup_Size_X"])
        t = 0
        for name, grid, us in launches:
            w.writerow([name, t, t + int(us * 1000), grid, 256])
            t += int(us * 1000) + 500
    return str(path)


def _tuned_run(timed):
    """Trials of four sweep shapes and the split step, twice six launches each,
    then the timed region on the split step."""
    out = []
    for _ in range(2):
        for grid in (1024, 2048, 4096, 8192):
            out += [(SWEEP, grid, 1100.0)] * 6
        out += [(MOMENTS, 512, 500.0), (COLLIDE, 512, 520.0)] * 6
    return out + [(MOMENTS, 512, 420.0), (COLLIDE, 512, 440.0)] * timed


def test_forms_summary_skips_trials(tmp_path):
    t = _trace(tmp_path / "t.csv", _tuned_run(40) + [(PAIRS, 64, 1000.0)] * 40)
    txt = profiling.forms_summary(t, str(tmp_path / "o.md"), 40, "cmd")
    assert "k_step_fusedIDF16_" not in txt
    assert "| 420.0 | 420.0 | 420.0 |" in txt and "| 440.0 | 440.0 | 440.0 |" in txt
    assert "FP16 pairs, split: moments" in txt and "FP32 pairs |" in txt


def test_trace_summary_refuses_a_kernel_without_a_timed_region(tmp_path):
    t = _trace(tmp_path / "t.csv", [(PAIRS, g, 1000.0) for g in (64, 128, 256) for _ in range(6)])
    for region in ("first", "last"):
        with pytest.raises(SystemExit):
            profiling.trace_summary(t, str(tmp_path / "o.md"), "k_step_fused", 20, "cmd", region)
    t = _trace(tmp_path / "t.csv", [(PAIRS, 64, 1000.0)] * 6 + [(PAIRS, 128, 900.0)] * 20)
    txt = profiling.trace_summary(t, str(tmp_path / "o.md"), "k_step_fused", 20, "cmd", "first")
    assert "average duration: 900.0 us" in txt
