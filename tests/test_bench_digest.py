"""CPU: counters recorded for a kernel stay good while sources that it does not
include change, and are dropped when one of its own does."""
import json
import os
import shutil

import bench

CSRC = os.path.join(bench.ROOT, "paper_1912_06680_amd", "csrc")


def _touch(path):
    with open(path, "a") as fh:
        fh.write("// changed\n")


def test_a_kernels_digest_covers_its_file_and_headers_only(tmp_path):
    d = str(tmp_path / "csrc")
    shutil.copytree(CSRC, d)
    before = {k: bench.kernel_digest(k, d) for k in bench.SITE_SOURCES}
    assert before == {k: bench.kernel_digest(k) for k in bench.SITE_SOURCES}
    _touch(os.path.join(d, "sample.hip"))
    assert before == {k: bench.kernel_digest(k, d) for k in bench.SITE_SOURCES}
    _touch(os.path.join(d, "gemm_dma.h"))  # through gemm_plan.h, gemm_f32.h
    after = {k: bench.kernel_digest(k, d) for k in bench.SITE_SOURCES}
    assert after["lstm_fwd_gemm"] != before["lstm_fwd_gemm"]
    assert after["adam_step"] == before["adam_step"] and after["gae"] == before["gae"]
    _touch(os.path.join(d, "common.h"))
    assert all(bench.kernel_digest(k, d) != after[k] for k in bench.SITE_SOURCES)


def test_counters_of_an_unchanged_kernel_are_used(tmp_path):
    k = {"fetch_bytes_per_launch": 1, "write_bytes_per_launch": 2, "source_digest": bench.kernel_digest("adam_step")}
    t = {"source_digest": "0" * 64, "kernels": {"adam_step": k, "gae": dict(k)}}
    p = tmp_path / "t.json"
    p.write_text(json.dumps(t))
    assert bench.measured_traffic("adam_step", str(p)) == 3
    assert bench.measured_traffic("gae", str(p)) is None  # another kernel's sources
