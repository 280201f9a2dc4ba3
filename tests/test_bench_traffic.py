"""bench.py reports counted traffic only for the launches it was counted on: that workload,
that site, and the kernel source the summary names."""
import hashlib

import bench


def test_traffic_only_of_the_counted_launches(tmp_path, monkeypatch):
    src, summary = tmp_path / "kernel.hpp", tmp_path / "counters.md"
    src.write_text("kernel\n")
    digest = hashlib.sha256(src.read_bytes()).hexdigest()[:16]
    summary.write_text(f"traffic_bytes_per_launch: 1.5e+09\nkernel_source_sha256_16: {digest}\n")
    monkeypatch.setattr(bench, "PROFILE_FILES",
                        {("llama8b_like", "prefill_gu"): (str(summary), (str(src),))})
    assert bench.measured_traffic("llama8b_like", "prefill_gu") == 1.5e9
    assert bench.measured_traffic("small_bf16", "prefill_gu") is None
    assert bench.measured_traffic("llama8b_like", "prefill_qkv") is None
    src.write_text("another kernel\n")
    assert bench.measured_traffic("llama8b_like", "prefill_gu") is None


def test_named_summaries_exist():
    from paper_2609_38795_amd import workloads
    import os
    for (workload, _), (path, srcs) in bench.PROFILE_FILES.items():
        assert workload in workloads.WORKLOADS
        for f in (path, *srcs):
            assert os.path.exists(os.path.join(bench.ROOT, f))
