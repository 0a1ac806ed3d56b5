"""Which committed profile summaries the benchmark's roofline takes."""
import pytest

import bench

TRACE = """Kernel trace.

kernel_source_digest: {digest}
schedule: {schedule}

  kernel                                          calls   total ms    avg us       %   min us   max us
  void sim::k_step<2, 3>(sim::Dev const*, sim::    3600      51.73     14.37   48.19     7.52    19.80
"""


@pytest.mark.parametrize("digest,schedule,taken", [(None, "16,8,16", True), (None, "8,8,8", False),
                                                   ("0123456789abcdef", "16,8,16", False)])
def test_summaries_of_other_schedules_or_kernels_are_left(tmp_path, monkeypatch, digest, schedule, taken):
    digest = digest or bench.kernel_source_digest()
    monkeypatch.setattr(bench, "kernel_source_digest", lambda: digest if taken or schedule == "8,8,8" else "current")
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "step_kernels_w_kernel_trace.txt").write_text(TRACE.format(digest=digest, schedule=schedule))
    (tmp_path / "profiles" / "k_step_w_hbm_traffic.txt").write_text(
        f"kernel_source_digest: {digest}\nschedule: {schedule}\nhbm_bytes_per_launch: 29200000\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.rocprof_avg_us("k_step", "w", [16, 8, 16]) == (14.37 if taken else None)
    assert bench.measured_traffic("k_step", "w", (16, 8, 16)) == (29200000 if taken else None)
    assert bench.rocprof_avg_us("k_step", "other", [16, 8, 16]) is None
