"""bench.py reports counter traffic only for the kernels that the committed counter profile measured (no GPU)."""
import bench


def test_traffic_of_other_kernel_sources_is_not_reported(tmp_path, monkeypatch):
    label = "linear_packed 300x10240x1280 geglu ln"
    text = "kernel_sources_digest %s\ntraffic_per_step_bytes gemm 1000\ntraffic_per_launch_bytes 250 " + label + "\n"
    profile = tmp_path / "traffic.md"
    monkeypatch.setattr(bench, "TRAFFIC_PROFILE", str(profile))
    profile.write_text(text % bench.kernel_sources_digest())
    assert bench.traffic_from_profile(cls="gemm") == 1000.0 and bench.traffic_from_profile(kernel=label) == 250.0
    for stale in (text % "0123456789abcdef", text.split("\n", 1)[1]):
        profile.write_text(stale)
        assert bench.traffic_from_profile(cls="gemm") is None and bench.traffic_from_profile(kernel=label) is None
