"""bench.py names the sweep kernel that the tuned launch shape runs and attaches
the measured traffic of that shape, not of another one's."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


@pytest.mark.parametrize("shape,kernel,traffic", [
    ((2, 256, 0, 4), "k_sweep_tile", 5.5e9),
    ((4, 768, 0, 0), "k_sweep", 6.1e9),
    ((4, 768, 8, 0), "k_sweep", None),  # not in this summary
    ((1, 768, 0, 2), "k_sweep_tile", 5.4e9),
])
def test_kernel_and_traffic_follow_the_shape(tmp_path, monkeypatch, shape, kernel, traffic):
    source, summary = tmp_path / "s.hip", tmp_path / "s.md"
    source.write_text("int x;\n")
    summary.write_text("(traffic_bytes_per_launch[tile 2x4]: 5.5e9)\n(traffic_bytes_per_launch[tile 1x2]: 5.4e9)\n"
                       "(traffic_bytes_per_launch[pencils 4]: 6.1e9)\n(kernel_source_sha256_prefix: %s)\n"
                       % bench.kernel_source_digest(str(source))[:16])
    monkeypatch.setitem(bench.TRAFFIC_SUMMARY, "k_sweep", (str(summary), str(source)))
    name, key = bench.sweep_kernel(shape)
    assert name == kernel
    assert bench.measured_traffic("k_sweep", "cfg3", "fp32", key) == traffic
