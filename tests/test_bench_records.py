"""The benchmark's record of the per-step FP32 path: rates that the card can reach."""
import pytest

import bench


def test_per_step_record_states_the_rate_of_the_arithmetic():
    N, M, n_md = 9216, 27648, 256
    fastest = 24.0 * N * M * n_md / bench.PEAK_FP32_VALU_FLOPS * 1e3      # ms: every FMA at the vector peak
    r = bench.per_step_record(N, M, n_md, 2e-3 * fastest, fastest)
    assert r["kernel_frac"] == pytest.approx(1.0) and r["kernel_TFLOPs"] == pytest.approx(bench.PEAK_FP32_VALU_FLOPS / 1e12)
    assert r["value"] == pytest.approx(N * M * n_md / (2e-3 * fastest)) and r["md_steps"] == n_md
    # four steps to a pass over the basis: 12 B per atom, mode and step would be more than the memory delivers
    assert not [k for k in r if "GBps" in k]
    assert bench.per_step_record(N, M, n_md, 1.0, 0.0)["kernel_frac"] is None
